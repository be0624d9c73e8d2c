// Ring kernel of the bf16 GEMM family: small tiles, K slices of 64 loaded with global_load_lds_dwordx4 into a deep
// ring of LDS stages.
//
// Where it is used: products whose tiles are few or short, i.e. a few thousand rows or columns of a few hundred.  What
// bounds those is not a pipe but latency: with the slices of a tile fetched one ahead through registers, every
// slice costs a memory round trip (measured on [788 x 768 x 3072]: 0.94 us per slice of 64).  Here RING slices are
// in flight per workgroup, without holding registers, and the tiles are small enough that the launch has a
// workgroup for every CU.
//
// One workgroup computes BM x BN: four waves (2 x 2) a tile of 64 x 64, eight waves one of 64 x 128, 128 x 64 or 128 x 128, which
// read a half and a quarter less of the operands (a CU takes in about 100 bytes per ns from the L2 while all do, 0.16 us for
// the 16 KB of a 64 x 64 slice) where they still leave a workgroup for most CUs.  Per slice t: wait for the loads of slice t + 1
// (s_waitcnt vmcnt counts loads in order, younger slices stay in flight), one barrier, request slice t + RING into the
// stage of slice t, whose fragments every wave holds in registers by then, read the fragments of slice t + 1, multiply
// slice t.  LDS layouts, bank swizzles and the exchanged MFMA
// operands are those of gemm_bf16_kernels.h; with rows of 64 elements (128 bytes) a transposed operand is swizzled by
// ((k >> 1) & 1) << 2 instead, two k-rows filling one 256-byte bank span.
// Ragged K needs no predicate on the data path: in the last slice a lane whose piece lies beyond the end reads a block
// of zeros instead.  A piece of a row-major operand is 8 k values, so its columns K .. round8(K) - 1 are read and multiplied, by
// zeros if the other operand is transposed and by that one's own if it is row-major too: such padding has to be finite, and zero
// in one of two row-major operands (as in every other tile of this family).  The same block stands in for
// the pixels outside the image of an implicit convolution (CONV = 1: operand A is gathered, CONV = 2: operand B of a weight
// gradient is, over any number of output pixels; geometry from the launch arguments, see gemm_pp_kernel).
#pragma once
#include "gemm_bf16_kernels.h"

namespace et {
namespace gemm {

// the product of a launch: its arguments, or a job of a group as such
template <bool CONV>
__device__ __forceinline__ const Params& ring_product(const Params& p, const Params&, int) { return p; }
template <bool CONV>
__device__ __forceinline__ const Params& ring_product(const GroupParams<CONV>& p, Params& g, int job) {
  const auto& j = p.job[job];
  g.A = j.A; g.B = j.B; g.M = j.M; g.N = j.N; g.K = j.K; g.lda = j.lda; g.ldb = j.ldb;
  g.split_k = j.split; g.k_chunk = j.k_chunk; g.z_inner = 1;
  g.sAo = g.sAi = g.sBo = g.sBi = g.sCo = g.sCi = 0;
  g.C = j.C;
  if constexpr (CONV) { g.cH = j.cH; g.cW = j.cW; g.cC = j.cC; g.cT = j.cT; g.cS = j.cS; g.cHo = j.cHo; g.cWo = j.cWo; }
  return g;
}

// GROUP: the weight gradients of a whole backward pass in one launch: one workgroup per unit, the units with the longest chunks first.  What it is
// for: a gradient of its own is a launch of 4 - 15 us that fills the chip once with chunks of the reduction, and a second launch adds them up;
// together the gradients have tiles enough with few chunks or none.
template <int BM, int BN, int WGM, int WGN, int RING, bool AT, bool BT, int EPI, int CONV = 0, bool GROUP = false>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_ring_kernel(std::conditional_t<GROUP, GroupParams<CONV == 2>, Params> args) {
  static_assert(!GROUP || (AT && BT && EPI == E_PARTIAL && CONV != 1), "groups of weight gradients");
  constexpr int NW = WGM * WGN;
  constexpr int TM = BM / WGM, TN = BN / WGN;
  constexpr int MI = TM / 32, NI = TN / 32;
  constexpr int A_BYTES = BM * PBK * 2, B_BYTES = BN * PBK * 2, STAGE = A_BYTES + B_BYTES;
  constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = B_BYTES / 1024 / NW, LOADS = A_LOADS + B_LOADS;
  static_assert(A_LOADS * 1024 * NW == A_BYTES && B_LOADS * 1024 * NW == B_BYTES, "tile/waves mismatch");
  static_assert(CONV != 1 || (!AT && !BT), "implicit convolution, forward: row-major operands");
  static_assert(CONV != 2 || (AT && BT), "implicit convolution, weight gradient: both operands reduce over rows");
  constexpr int EPI_BYTES = NW * epi_wave_bytes<TN>();
  constexpr int SMEM = RING * STAGE > EPI_BYTES ? RING * STAGE : EPI_BYTES;
  static_assert(RING >= 2 && RING <= 5 && SMEM <= 160 * 1024, "LDS ring");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave / WGN, wave_n = wave % WGN;
  int m0, n0, z, job = 0, unit = 0;
  if constexpr (GROUP) {
    unit = group_unit((int)blockIdx.x, 1024, args.units);
    job = group_job<CONV == 2>(args, unit);
  }
  Params from_job;
  const Params& g = ring_product<CONV == 2>(args, from_job, job);
  if constexpr (GROUP) group_tile<BM, BN>(g.M, g.N, unit - args.job[job].unit0, m0, n0, z);
  else tile_coords<BM, BN>(g, m0, n0, z);
  const bf16* A;
  const bf16* B;
  long long c_off;
  int k_begin, k_end;
  batch_offsets(g, z, A, B, c_off, k_begin, k_end);
  const int nk = (k_end - k_begin + PBK - 1) / PBK;
  // (k_end > 0 in every chunk; rows of a row-major operand are readable up to K rounded up to 8)
  const int rem_t = k_end - k_begin - (nk - 1) * PBK;                                              // k values of the last slice
  const int rem_r = min((g.K + 7) & ~7, (k_end + 7) & ~7) - k_begin - (nk - 1) * PBK;

  // implicit convolutions.  CONV 1: output pixel of each piece's row (input coordinates of its centre tap); tap and channel of
  // the next slice, uniform.  CONV 2: per piece (dy + 1) << 26 | (dx + 1) << 24 | ho << 12 | wo for its tap and the output
  // pixel of its k-row (the pixel advances by 64 per slice), and the tap's element offset
  const int cS = g.cS, cT = g.cT, cHo = g.cHo, cWo = g.cWo, ssh = g.cS >> 1;
  int coh[CONV == 1 ? A_LOADS : 1], cow[CONV == 1 ? A_LOADS : 1];
  int bpix[CONV == 2 ? B_LOADS : 1], boff[CONV == 2 ? B_LOADS : 1];
  int c_dy = 0, c_dx = 0, c_sub = 0;
  long long c_off_a = 0;

  // per-lane global source of each of this wave's 1 KiB pieces (slice 0), and the k index within a slice it starts at
  const bf16* ga[A_LOADS];
  const bf16* gb[B_LOADS];
  int ka[A_LOADS], kb[B_LOADS];
  auto swz_t = [](int rows, int k) { return rows == 64 ? ((k >> 1) & 1) << 2 : (k & 3) << 2; };
#pragma unroll
  for (int i = 0; i < A_LOADS; i++) {
    const int q = wave * A_LOADS + i;
    if (!AT) {   // 8 rows x 128 B; 16-byte chunk c of row r sits at chunk position c ^ ((r >> 1) & 7)
      const int row = q * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
      const int m = min(m0 + row, g.M - 1);
      ka[i] = chunk * 8;
      if (CONV == 1) {
        const int wo = m % cWo, t = m / cWo, ho = t % cHo, img = t / cHo;
        cow[CONV == 1 ? i : 0] = wo * cS;
        coh[CONV == 1 ? i : 0] = ho * cS;
        ga[i] = A + ((long long)(img * g.cH + ho * cS) * g.cW + wo * cS) * g.cC + chunk * 8;
      } else {
        ga[i] = A + (long long)m * g.lda + k_begin + chunk * 8;
      }
    } else {     // [64 k-rows][BM]; chunk j of k-row k sits at chunk position j ^ swz_t(k)
      constexpr int CR = BM / 8;
      const int pos = q * 64 + lane;
      const int k = pos / CR, j = (pos % CR) ^ swz_t(BM, k);
      int gi = m0 + j * 8;
      if (gi + 8 > ((g.M + 7) & ~7)) gi = 0;
      ka[i] = k;
      ga[i] = A + (long long)(k_begin + k) * g.lda + gi;
    }
  }
#pragma unroll
  for (int i = 0; i < B_LOADS; i++) {
    const int q = wave * B_LOADS + i;
    if (!BT) {
      const int row = q * 8 + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
      kb[i] = chunk * 8;
      gb[i] = B + (long long)min(n0 + row, g.N - 1) * g.ldb + k_begin + chunk * 8;
    } else {
      constexpr int CR = BN / 8;
      const int pos = q * 64 + lane;
      const int k = pos / CR, j = (pos % CR) ^ swz_t(BN, k);
      int gj = n0 + j * 8;
      if (gj + 8 > ((g.N + 7) & ~7)) gj = 0;
      kb[i] = k;
      if (CONV == 2) {   // column gj = (tap, channel) of the matrix; N = taps^2 cC and cC are multiples of 8
        const int tap = gj / g.cC, ch = gj % g.cC;
        const int dy = tap / cT - (cT >> 1), dx = tap % cT - (cT >> 1);
        const int pix = min(k_begin + k, g.K - 1);   // (never read from beyond the last pixel)
        const int wo = pix % cWo, t = pix / cWo, ho = t % cHo, img = t / cHo;
        bpix[CONV == 2 ? i : 0] = ((dy + 1) << 26) | ((dx + 1) << 24) | (ho << 12) | wo;
        boff[CONV == 2 ? i : 0] = (dy * g.cW + dx) * g.cC;
        gb[i] = B + ((long long)(img * g.cH + ho * cS) * g.cW + wo * cS) * g.cC + ch;
      } else {
        gb[i] = B + (long long)(k_begin + k) * g.ldb + gj;
      }
    }
  }
  if (CONV == 1) {   // tap and channel of the first slice to load
    const int tap0 = k_begin / g.cC;
    c_sub = k_begin % g.cC;
    c_dy = tap0 / cT - (cT >> 1);
    c_dx = tap0 % cT - (cT >> 1);
    c_off_a = (long long)(c_dy * g.cW + c_dx) * g.cC + c_sub;
  }
  const long long a_step = AT ? (long long)PBK * g.lda : PBK;
  const long long b_step = BT ? (long long)PBK * g.ldb : PBK;
  const unsigned lds0 = (unsigned)(unsigned long long)(__attribute__((address_space(3))) unsigned char*)smem;
  const bf16* const zeros = (const bf16*)kZeroBlock;
  // CONV 2: the move by 64 output pixels, (image, ho, wo) += (b_sb, b_sh, b_sw) with carries, as element distances
  const int b_sw = CONV == 2 ? PBK % cWo : 0, b_sh = CONV == 2 ? (PBK / cWo) % cHo : 0, b_sb = CONV == 2 ? PBK / (cWo * cHo) : 0;
  const int b_d0 = CONV == 2 ? ((b_sb * g.cH + (b_sh << ssh)) * g.cW + (b_sw << ssh)) * g.cC : 0;
  const int b_dw = CONV == 2 ? ((g.cW - cWo) << ssh) * g.cC : 0, b_dh = CONV == 2 ? (g.cH - (cHo << ssh)) * g.cW * g.cC : 0;

  // one slice into `stage`; lim_a, lim_b: how many of its 64 k values exist (64: no test)
  auto issue_some = [&](int stage, auto full_tag, int lim_a, int lim_b) {
    constexpr bool FULL = decltype(full_tag)::value;
    const unsigned sa = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + wave * A_LOADS * 1024);
    const unsigned sb = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + A_BYTES + wave * B_LOADS * 1024);
#pragma unroll
    for (int i = 0; i < A_LOADS; i++) {
      const bf16* p = ga[i];
      bool ok = FULL || ka[i] < lim_a;
      if (CONV == 1) {
        ok = (unsigned)(coh[CONV == 1 ? i : 0] + c_dy) < (unsigned)g.cH && (unsigned)(cow[CONV == 1 ? i : 0] + c_dx) < (unsigned)g.cW;
        p += c_off_a;
      } else {
        ga[i] += a_step;
      }
      dma16(ok ? p : zeros, sa + i * 1024);
    }
    if (CONV == 1) {
      c_sub += PBK;
      if (c_sub == g.cC) {
        c_sub = 0;
        if (++c_dx > (cT >> 1)) { c_dx = -(cT >> 1); c_dy++; }
      }
      c_off_a = (long long)(c_dy * g.cW + c_dx) * g.cC + c_sub;
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; i++) {
      const bf16* p = gb[i];
      bool ok = FULL || kb[i] < lim_b;
      if (CONV == 2) {
        const int k = CONV == 2 ? i : 0;
        const int dy = (bpix[k] >> 26) - 1, dx = ((bpix[k] >> 24) & 3) - 1;
        int h = (bpix[k] >> 12) & 4095, w = bpix[k] & 4095;
        ok = ok && (unsigned)((h << ssh) + dy) < (unsigned)g.cH && (unsigned)((w << ssh) + dx) < (unsigned)g.cW;
        p += boff[k];
        int delta = b_d0;
        w += b_sw;
        h += b_sh;
        if (w >= cWo) { w -= cWo; h++; delta += b_dw; }
        if (h >= cHo) { h -= cHo; delta += b_dh; }
        gb[i] += delta;
        bpix[k] = (bpix[k] & ~0xffffff) | (h << 12) | w;
      } else {
        gb[i] += b_step;
      }
      dma16(ok ? p : zeros, sb + i * 1024);
    }
  };
  auto issue_full = [&](int stage) { issue_some(stage, std::true_type(), PBK, PBK); };
  auto issue = [&](int sl, int stage) {
    if (sl + 1 < nk || rem_t == PBK) issue_full(stage);
    else issue_some(stage, std::false_type(), AT ? rem_t : rem_r, BT ? rem_t : rem_r);   // the ragged last slice
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; mi++)
#pragma unroll
    for (int ni = 0; ni < NI; ni++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[mi][ni][r] = 0.f;

  const int l32 = lane & 31, khalf = lane >> 5;
  const int grp16 = lane >> 4, r16 = lane & 15;
  const int tr_col = (grp16 & 1) * 16 + 4 * (r16 & 3);
  const int tr_krow = (grp16 >> 1) * 8 + (r16 >> 2);   // k-rows tr_krow and tr_krow + 4: the same swizzle for both

  auto load_a = [&](const unsigned char* st, int ks, int mi) -> bf16x8 {
    const int rbase = wave_m * TM + mi * 32;
    if (!AT) {
      const int row = rbase + l32, chunk = ks * 2 + khalf;
      return *(const bf16x8*)(st + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    } else {
      const int col = rbase + tr_col;
      const unsigned char* p = st + (ks * 16 + tr_krow) * (BM * 2) + (((col >> 3) ^ swz_t(BM, tr_krow)) << 4) + ((col >> 2) & 1) * 8;
      bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * (BM * 2));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  auto load_b = [&](const unsigned char* st, int ks, int ni) -> bf16x8 {
    const unsigned char* sb = st + A_BYTES;
    const int rbase = wave_n * TN + ni * 32;
    if (!BT) {
      const int row = rbase + l32, chunk = ks * 2 + khalf;
      return *(const bf16x8*)(sb + row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4));
    } else {
      const int col = rbase + tr_col;
      const unsigned char* p = sb + (ks * 16 + tr_krow) * (BN * 2) + (((col >> 3) ^ swz_t(BN, tr_krow)) << 4) + ((col >> 2) & 1) * 8;
      bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 4 * (BN * 2));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };

  // wait until slice `sl` has landed: up to `most` younger slices stay in flight
  auto wait_slice = [&](int sl, auto most_tag) {
    constexpr int MOST = decltype(most_tag)::value;
    static_assert(MOST <= 4 && MOST * LOADS <= 63, "vmcnt");
    const int younger = min(MOST, nk - 1 - sl);
    if (younger == MOST) { wait_vmcnt<MOST * LOADS>(); return; }
    if (MOST > 3 && younger == 3) wait_vmcnt<3 * LOADS>();
    else if (MOST > 2 && younger == 2) wait_vmcnt<2 * LOADS>();
    else if (MOST > 1 && younger == 1) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
  };
  // workgroup barrier at which this wave's LDS reads have arrived and its share of the awaited slice has landed
  auto slice_barrier = [&]() {
    // (the builtin, not inline assembly: the compiler then knows that the fragments need no further wait)
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    block_barrier();
  };
  constexpr int KS = PBK / 16;
  struct Frags { bf16x8 a[KS][MI], b[KS][NI]; };
  auto read_frags = [&](int stage, Frags& f) {
    const unsigned char* st = smem + stage * STAGE;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
#pragma unroll
      for (int mi = 0; mi < MI; mi++) f.a[ks][mi] = load_a(st, ks, mi);
#pragma unroll
      for (int ni = 0; ni < NI; ni++) f.b[ks][ni] = load_b(st, ks, ni);
    }
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int mi = 0; mi < MI; mi++)
#pragma unroll
        for (int ni = 0; ni < NI; ni++)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ks][ni], f.a[ks][mi], acc[mi][ni], 0, 0, 0);
  };

#pragma unroll
  for (int sl = 0; sl < RING; sl++)
    if (sl < nk) issue(sl, sl);
  int stage = 0;                    // stage of slice kt
  Frags f0, f1;
  wait_slice(0, std::integral_constant<int, RING - 1>());
  block_barrier();
  read_frags(0, f0);
  // one slice: its fragments are in `cur`; the next slice's are requested into `nxt` before the multiplication, and the
  // stage just read (every wave's fragments of it have arrived at the barrier) receives the slice RING ahead
  auto next_stage = [&]() { stage = stage + 1 == RING ? 0 : stage + 1; };
  auto step_full = [&](Frags& cur, Frags& nxt) {   // not among the last RING + 1 slices: no conditions
    wait_vmcnt<(RING - 2) * LOADS>();
    slice_barrier();
    issue_full(stage);
    next_stage();
    read_frags(stage, nxt);
    __builtin_amdgcn_sched_barrier(0);   // the reads travel under the multiplication
    mma(cur);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&](int kt, Frags& cur, Frags& nxt) {
    if (kt + 1 < nk) {
      wait_slice(kt + 1, std::integral_constant<int, RING - 2>());
      slice_barrier();
      if (kt + RING < nk) issue(kt + RING, stage);
      next_stage();
      read_frags(stage, nxt);
    }
    mma(cur);
  };
  int kt = 0;
  for (; kt + RING + 2 < nk; kt += 2) {
    step_full(f0, f1);
    step_full(f1, f0);
  }
  for (; kt < nk; kt += 2) {
    step(kt, f0, f1);
    if (kt + 1 < nk) step(kt + 1, f1, f0);
  }
  __syncthreads();   // every wave is done with the stages before they are reused for the epilogue
  wave_epilogue<EPI, MI, NI>(g, acc, smem + wave * epi_wave_bytes<TN>(), m0 + wave_m * TM, n0 + wave_n * TN, c_off, lane);
}

LaunchFn ring_64x64(bool a_t, bool b_t, int epi);
LaunchFn ring_64x64_deep(bool a_t, bool b_t, int epi);   // five slices in flight, or null
LaunchFn ring_64x128(bool a_t, bool b_t, int epi);
LaunchFn ring_128x128(bool a_t, bool b_t, int epi);
LaunchFn ring_conv_64x64(int epi);
LaunchFn ring_conv_64x128(int epi);
LaunchFn ring_conv_128x64(int epi);
LaunchFn ring_conv_128x128(int epi);
LaunchFn ring_convdw_64x64(int epi);
LaunchFn ring_convdw_64x128(int epi);
LaunchFn ring_convdw_128x64(int epi);

}  // namespace gemm
}  // namespace et
