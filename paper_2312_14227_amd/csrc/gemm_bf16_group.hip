// The weight gradients of a backward pass in one launch per kind of kernel: plan, instantiations of the grouped kernels (see
// gemm_bf16_direct.h, gemm_bf16_ring.h), and the launch that adds the chunks of those that were split.
#include <algorithm>
#include <cmath>
#include <vector>

#include "gemm_bf16_direct.h"
#include "gemm_bf16_ring.h"

namespace et {
namespace gemm {
namespace {

template <int MI>
hipError_t launch(const GroupParams<false>& p, int grid, hipStream_t s) {
  hipLaunchKernelGGL((gemm_direct_kernel<MI, true, true, E_PARTIAL, true>), dim3(grid), dim3(512), 0, s, p);
  return hipGetLastError();
}
template <int BM, int BN, int WGM, int WGN, bool GATHERED>
hipError_t launch_ring(const GroupParams<GATHERED>& p, hipStream_t s) {
  hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WGM, WGN, 3, true, true, E_PARTIAL, GATHERED ? 2 : 0, true>), dim3(p.units), dim3(WGM * WGN * 64), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t direct_group(int rows, const GroupParams<false>& p, int grid, hipStream_t s) {
  return rows == 256 ? launch<4>(p, grid, s) : rows == 192 ? launch<3>(p, grid, s) : launch<2>(p, grid, s);
}
hipError_t ring_group_64x64(const GroupParams<false>& p, hipStream_t s) { return launch_ring<64, 64, 2, 2, false>(p, s); }
hipError_t ring_group_64x128(const GroupParams<false>& p, hipStream_t s) { return launch_ring<64, 128, 2, 4, false>(p, s); }
hipError_t ring_group_conv_64x64(const GroupParams<true>& p, hipStream_t s) { return launch_ring<64, 64, 2, 2, true>(p, s); }
hipError_t ring_group_conv_64x128(const GroupParams<true>& p, hipStream_t s) { return launch_ring<64, 128, 2, 4, true>(p, s); }

}  // namespace gemm
}  // namespace et

namespace et {
namespace {

constexpr int SLICE = gemm::PBK;

struct ReduceJob {
  const float4* part;
  float4* out;
  int n4, splits, wide, block0;
};
constexpr int MAX_REDUCE = DW_GROUP_MAX;   // (kernel arguments: 32 bytes each)
struct ReduceJobs {
  int n;
  ReduceJob job[MAX_REDUCE];
};

// out[i] = sum over chunks, in ascending order; many chunks of few outputs: 16 lanes share an output vector, lane g adds the chunks g, g + 16, ..,
// then the 16 sums are added in lane order (both as a split product on its own does)
__global__ __launch_bounds__(256) void group_reduce_kernel(ReduceJobs jobs) {
  __shared__ float4 sh[16][16];
  int lo = 0, hi = jobs.n - 1;   // the job this workgroup belongs to: the last with block0 <= blockIdx.x
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs.job[mid].block0 <= (int)blockIdx.x) lo = mid;
    else hi = mid - 1;
  }
  const ReduceJob j = jobs.job[lo];
  const int block = (int)blockIdx.x - j.block0;
  const int o = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const int i = j.wide ? block * 16 + o : block * 256 + (int)threadIdx.x;
  const int first = j.wide ? grp : 0, step = j.wide ? 16 : 1;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < j.n4) {
#pragma unroll 4
    for (int z = first; z < j.splits; z += step) {
      const float4 p = j.part[(size_t)z * j.n4 + i];
      s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
  }
  if (!j.wide) {
    if (i < j.n4) j.out[i] = s;
    return;
  }
  sh[grp][o] = s;
  __syncthreads();
  if (grp == 0 && i < j.n4) {
    float4 t = sh[0][o];
    for (int k = 1; k < 16; k++) {
      const float4 p = sh[k][o];
      t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    j.out[i] = t;
  }
}

typedef DwGroupLaunch Launch;
typedef DwGroupLaunch::Part Planned;

inline int slices_of(const DwJob& j) { return (j.K + SLICE - 1) / SLICE; }
inline long long tiles_of(const DwJob& j, int bm, int bn) { return (long long)((j.M + bm - 1) / bm) * ((j.N + bn - 1) / bn); }
inline Planned part_of(const DwJob& j, int index, int bm, int bn) {
  const int sl = slices_of(j), per = (sl + j.split - 1) / j.split;
  return {index, (sl + per - 1) / per, per, tiles_of(j, bm, bn)};   // (no empty chunks)
}
inline void longest_first(std::vector<Planned>& parts) {
  std::stable_sort(parts.begin(), parts.end(), [](const Planned& a, const Planned& b) { return a.per > b.per; });
}

// Ring tiles: a workgroup per unit, dealt as CUs become free, longest chunks first.  us per slice with several workgroups per CU, which grows with the
// length of the chunks and the number of units per CU (operand re-reads: [1536 x 384] and the like over 4616 rows, 2600 units, 0.46 us per
// slice of a 64 x 128 tile), with one, and per unit.
Launch plan_ring(const DwJob* jobs, const std::vector<int>& which, bool gathered) {
  struct Tile { int bm, bn; double loaded, length, rounds, solo, fixed; };
  static const Tile plain[2] = {{64, 64, 0.116, 0.00047, 0.0122, 0.25, 0.5}, {64, 128, 0.179, 0.00069, 0.0228, 0.36, 1.0}};
  static const Tile conv[2] = {{64, 64, 0.17, 0.00047, 0.0122, 0.365, 0.5}, {64, 128, 0.24, 0.00069, 0.0228, 0.46, 1.0}};
  Launch best;
  best.cost = 1e30;
  for (const Tile& t : gathered ? conv : plain) {
    Launch l;
    l.gathered = gathered; l.bm = t.bm; l.bn = t.bn;
    double units = 0.0, work = 0.0;
    int longest = 0;
    for (int i : which) {
      l.parts.push_back(part_of(jobs[i], i, t.bm, t.bn));
      units += (double)l.parts.back().tiles * l.parts.back().split;
      longest = std::max(longest, l.parts.back().per);
    }
    const double rounds = std::min(12.0, units / 256.0);
    for (const Planned& p : l.parts) work += (double)p.tiles * p.split * (p.per * (t.loaded + t.length * p.per + t.rounds * rounds) + t.fixed);
    l.cost = std::max(work / 256.0 + 0.5 * longest * t.loaded, longest * t.solo + t.fixed) + 3.0;
    if (l.cost < best.cost) best = l;
  }
  longest_first(best.parts);
  return best;
}

// Direct tiles: 256 resident workgroups take one unit per round, longest chunks first.  us per slice, more with all CUs at work, and per round.
Launch plan_direct(const DwJob* jobs, const std::vector<int>& which) {
  struct Tile { int bm; double slice, load, fixed; };
  static const Tile tile[3] = {{256, 0.833, 0.696, 5.4}, {192, 0.841, 0.419, 3.8}, {128, 0.765, 0.304, 2.4}};
  Launch best;
  best.cost = 1e30;
  for (const Tile& t : tile) {
    Launch l;
    l.direct = true; l.bm = t.bm; l.bn = 256;
    long long total = 0, at = 0;
    for (int i : which) {
      l.parts.push_back(part_of(jobs[i], i, t.bm, 256));
      total += l.parts.back().tiles * l.parts.back().split;
    }
    longest_first(l.parts);
    l.cost = 3.0;
    int longest = 0;   // of the round that is being filled
    for (const Planned& p : l.parts)
      for (long long n = p.tiles * p.split; n > 0;) {
        const long long here = std::min(n, 256 - at % 256);
        longest = std::max(longest, p.per);
        at += here;
        n -= here;
        if (at % 256 == 0 || at == total) {
          l.cost += longest * (t.slice + t.load * (at % 256 == 0 ? 1.0 : (at % 256) / 256.0)) + t.fixed;
          longest = 0;
        }
      }
    if (l.cost < best.cost) best = l;
  }
  return best;
}

template <bool CONV>
hipError_t run(const Launch& l, const DwJob* jobs, float* partials, size_t& used, ReduceJobs& reduce, int& reduce_blocks, hipStream_t s, int* launches) {
  typedef gemm::GroupParams<CONV> Group;
  for (size_t k = 0; k < l.parts.size();) {
    Group g;
    g.n = 0;
    g.units = 0;
    for (; k < l.parts.size() && g.n < Group::MAX; k++) {
      const Planned& p = l.parts[k];
      const DwJob& j = jobs[p.job];
      if (g.units + p.tiles * p.split >= (1ll << 30)) return hipErrorInvalidValue;
      auto& d = g.job[g.n++];
      d.A = j.A; d.B = j.B; d.C = j.C; d.M = j.M; d.N = j.N; d.K = j.K; d.lda = j.lda; d.ldb = j.ldb;
      d.split = p.split; d.k_chunk = p.per * SLICE; d.unit0 = g.units;
      if constexpr (CONV) {
        d.cH = j.conv_h; d.cW = j.conv_w; d.cC = j.conv_c; d.cT = j.conv_taps; d.cS = j.conv_stride;
        d.cHo = (j.conv_h - 1) / j.conv_stride + 1; d.cWo = (j.conv_w - 1) / j.conv_stride + 1;
      }
      g.units += (int)(p.tiles * p.split);
      if (p.split > 1) {
        ReduceJob& r = reduce.job[reduce.n++];
        r.n4 = (int)((long long)j.M * j.N / 4);
        r.splits = p.split;
        r.wide = p.split > 32;
        r.part = (const float4*)(partials + used);
        r.out = (float4*)j.C;
        r.block0 = reduce_blocks;
        reduce_blocks += r.wide ? (r.n4 + 15) / 16 : (r.n4 + 255) / 256;
        d.C = partials + used;
        used += (size_t)p.split * j.M * j.N;
      }
    }
    hipError_t e;
    if constexpr (CONV) e = l.bn == 128 ? gemm::ring_group_conv_64x128(g, s) : gemm::ring_group_conv_64x64(g, s);
    else if (l.direct) e = gemm::direct_group(l.bm, g, std::min(g.units, compute_units()), s);
    else e = l.bn == 128 ? gemm::ring_group_64x128(g, s) : gemm::ring_group_64x64(g, s);
    if (e != hipSuccess) return e;
    (*launches)++;
  }
  return hipSuccess;
}

}  // namespace

bool dw_group_takes(const DwJob& j) {
  const auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!j.A || !j.B || !j.C || !al(j.A) || !al(j.B) || !al(j.C) || j.M < 1 || j.N < 4 || j.K < 1 || j.split < 1 || (j.N & 3) || (j.lda & 7)) return false;
  if (j.lda < ((j.M + 7) & ~7) || (long long)j.M * j.N >= (1ll << 31)) return false;
  if (j.conv_c <= 0) return (j.ldb & 7) == 0 && j.ldb >= ((j.N + 7) & ~7);
  if ((j.conv_c & 7) || (j.conv_taps != 1 && j.conv_taps != 3) || (j.conv_stride != 1 && j.conv_stride != 2)) return false;
  if (j.conv_h < 1 || j.conv_w < 1 || j.conv_h > 4095 || j.conv_w > 4095 || j.N != j.conv_taps * j.conv_taps * j.conv_c) return false;
  const int ho = (j.conv_h - 1) / j.conv_stride + 1, wo = (j.conv_w - 1) / j.conv_stride + 1;
  return j.K % (ho * wo) == 0 && 2.0 * j.M * j.N * (double)j.K < 1.4e10;
}

hipError_t dw_group_plan(const DwJob* jobs, int n, DwGroupPlan& plan) {
  try {
    std::vector<long long> shapes;
    for (int i = 0; i < n; i++) {
      const DwJob& j = jobs[i];
      if (!dw_group_takes(j)) return hipErrorInvalidValue;
      for (long long v : {j.M, j.N, j.K, j.conv_c, j.lda, j.ldb, j.split}) shapes.push_back(v);
    }
    if (shapes == plan.shapes) return hipSuccess;
    plan.shapes.clear();
    plan.launches.clear();
    // plain gradients: the direct tiles for those that fill them, or everything on ring tiles, whichever is estimated to take less
    std::vector<int> large, small, plain, conv;
    for (int i = 0; i < n; i++) {
      if (jobs[i].conv_c > 0) {
        conv.push_back(i);
        continue;
      }
      plain.push_back(i);
      const bool fills = jobs[i].M >= 128 && jobs[i].N >= 192 && jobs[i].lda < (1 << 22) && jobs[i].ldb < (1 << 22);
      (fills ? large : small).push_back(i);
    }
    if (!plain.empty()) {
      Launch all = plan_ring(jobs, plain, false);
      if (!large.empty()) {
        Launch wide = plan_direct(jobs, large), few;
        if (!small.empty()) few = plan_ring(jobs, small, false);
        if (wide.cost + few.cost < all.cost) {
          plan.launches.push_back(wide);
          all = few;
        }
      }
      if (!all.parts.empty()) plan.launches.push_back(all);
    }
    if (!conv.empty()) plan.launches.push_back(plan_ring(jobs, conv, true));
    plan.cost.assign(n, 0.0);
    for (const Launch& l : plan.launches) {
      double units = 0.0;
      for (const Planned& p : l.parts) units += (double)p.tiles * p.split * (p.per + 2.0);
      for (const Planned& p : l.parts) plan.cost[p.job] = l.cost * (double)p.tiles * p.split * (p.per + 2.0) / units;
    }
    plan.shapes = shapes;
  } catch (const std::bad_alloc&) {
    return hipErrorOutOfMemory;
  }
  return hipSuccess;
}

hipError_t dw_group(const DwJob* jobs, int n, const DwGroupPlan& plan, float* partials, hipStream_t s, int* launches) {
  *launches = 0;
  if (n < 1 || n > DW_GROUP_MAX || (int)plan.cost.size() != n || !partials || (reinterpret_cast<uintptr_t>(partials) & 15)) return hipErrorInvalidValue;
  size_t used = 0;
  ReduceJobs reduce;
  reduce.n = 0;
  int blocks = 0;
  for (const Launch& l : plan.launches) {
    if (reduce.n + (int)l.parts.size() > MAX_REDUCE) return hipErrorInvalidValue;
    const hipError_t e = l.gathered ? run<true>(l, jobs, partials, used, reduce, blocks, s, launches)
                                    : run<false>(l, jobs, partials, used, reduce, blocks, s, launches);
    if (e != hipSuccess) return e;
  }
  if (reduce.n > 0) {
    hipLaunchKernelGGL(group_reduce_kernel, dim3(blocks), dim3(256), 0, s, reduce);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    (*launches)++;
  }
  return hipSuccess;
}

}  // namespace et
