// Dimension selection for the hierarchical exchange (HierMoE Section III-B/C, Eq.(1)-(6), Alg.1):
// per-level duplicate-free counts in one pass over the routing table, and the linear time model
// evaluated on the device so that the counts never travel to the host.
#include "hm_device.h"

namespace hm {

constexpr int kGroupThreads = 256;
constexpr int kMaxDepth = 4;

struct GroupParams {
  const int32_t *ids;
  const int32_t *expert_to_rank;
  int32_t T, K, E, G, depth;
  int32_t groups[kMaxDepth], per[kMaxDepth];   // groups of a level, ranks of a group
  int32_t *counts;   // [depth][64]
  int32_t *status;
};

__global__ __launch_bounds__(kGroupThreads) void group_clear_kernel(GroupParams p) {
  const int i = blockIdx.x * kGroupThreads + threadIdx.x;
  if (i < p.depth * kWave) p.counts[i] = 0;
  if (i == 0 && p.status) *p.status = 0;
}

// One lane per token: its rank mask is folded to one bit per group for every level, and lane j
// accumulates the popcount of the ballot over bit j (a token counts once per group).  What it waits for
// is the chain ids -> placement -> counts: a token's ids are loaded together, while the placement is
// staged in LDS (T=8192, K=8, four levels, kernel trace: 9.6 -> 6.2 us; it was one id after the other,
// each with its look-up in memory).  ALONE: the only workgroup (up to kAloneTokens tokens and
// more experts than can be staged); it stores the counts instead of adding to cleared ones, which saves the clearing launch.
constexpr int kAloneTokens = 1024;
template <int THREADS, bool ALONE>
__global__ __launch_bounds__(THREADS) void group_count_kernel(GroupParams p) {
  __shared__ int32_t block_cnt[kMaxDepth * kWave];
  __shared__ int8_t ranks[ALONE ? 1 : kStagedExperts];
  __shared__ int32_t bad;
  const bool staged = !ALONE && p.E <= kStagedExperts;
  const int64_t stride = (int64_t)gridDim.x * THREADS;
  int64_t t = (int64_t)blockIdx.x * THREADS + threadIdx.x;
  int id[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
  if (t < p.T) load_ids(p.ids + t * p.K, p.K, 0, id);   // on their way while the table is staged
  if (staged)
    for (int e = threadIdx.x; e < p.E; e += THREADS) ranks[e] = rank_code(p.G, p.expert_to_rank[e]);
  if (threadIdx.x < kMaxDepth * kWave) block_cnt[threadIdx.x] = 0;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  const int lane = lane_id();
  int mine[kMaxDepth] = {0, 0, 0, 0};
  bool my_bad = false;
  const int64_t rounds = ((int64_t)p.T + stride - 1) / stride;   // same for every lane: ballots stay convergent
  for (int64_t it = 0; it < rounds; ++it, t += stride) {
    uint64_t rm = 0;
    if (t < p.T) {
      for (int k0 = 0; k0 < p.K; k0 += 8) {
        if (it > 0 || k0 > 0) load_ids(p.ids + t * p.K, p.K, k0, id);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int g = staged ? staged_rank_of(ranks, p.E, id[j]) : rank_of(p.expert_to_rank, p.E, p.G, id[j]);
          my_bad = my_bad || g == -1;
          rm |= g >= 0 ? 1ull << g : 0ull;
        }
      }
    }
    if (__ballot(rm != 0) == 0) continue;
#pragma unroll
    for (int l = 0; l < kMaxDepth; ++l) {
      if (l >= p.depth) break;
      mine[l] += lanes_per_group(rm, p.groups[l], p.per[l]);
    }
  }
  if (my_bad) bad = 1;
#pragma unroll
  for (int l = 0; l < kMaxDepth; ++l)
    if (l < p.depth && lane < p.groups[l] && mine[l]) atomicAdd(&block_cnt[l * kWave + lane], mine[l]);
  __syncthreads();
  if ((int)threadIdx.x < p.depth * kWave) {
    const int v = block_cnt[threadIdx.x];
    if (ALONE) p.counts[threadIdx.x] = v;
    else if (v) atomicAdd(&p.counts[threadIdx.x], v);
  }
  if (threadIdx.x == 0) {
    if (ALONE) {
      if (p.status) *p.status = bad ? HM_ERR_BAD_ID : 0;
    } else if (bad) {
      flag(p.status, HM_ERR_BAD_ID);
    }
  }
}

// A workgroup owns seven groups of a level; SPREAD: for a part of the tokens, added to cleared outputs.
struct GroupOwners {
  int32_t first_block[kMaxDepth];        // of a level; beyond all blocks where there is no such level
  uint32_t per_recip16[kMaxDepth];       // ceil(2^16 / ranks of a group): exact for ranks (below 64)
  int32_t tokens;                        // of a workgroup, where they are spread
};
template <int W, bool SPREAD>
__global__ __launch_bounds__(kOwnerThreads) void group_owner_kernel(GroupParams p, GroupOwners o) {
  __shared__ uint8_t table[kOwnerMaxE + 2];
  int level = 0, block = (int)blockIdx.x, n = p.groups[0];
  uint32_t per_recip16 = o.per_recip16[0];
#pragma unroll
  for (int l = 1; l < kMaxDepth; ++l) {   // selects: a loop would wait for a load per level
    const bool from = (int)blockIdx.x >= o.first_block[l];
    level = from ? l : level;
    n = from ? p.groups[l] : n;
    per_recip16 = from ? o.per_recip16[l] : per_recip16;
    block = from ? (int)blockIdx.x - o.first_block[l] : block;
  }
  const int first = block * kOwnerGroups;
  const OwnerTokens t = owner_tokens<SPREAD>(p.ids, p.T, p.K, o.tokens);
  const int count = count_owned_groups<W>(t.ids, p.expert_to_rank, t.T, p.K, p.E, p.G, per_recip16, first, table);
  if (threadIdx.x >= kWave) return;
  const int lane = lane_id(), i = first + lane;
  if (SPREAD) {
    if (lane < kOwnerGroups && i < n && count) atomicAdd(&p.counts[level * kWave + i], count);
    if (blockIdx.x == 0 && lane == kOwnerGroups && count) flag(p.status, HM_ERR_BAD_ID);
    return;
  }
  // the last owner of a level clears what is behind its groups
  if (i < kWave && (lane < kOwnerGroups || first + kOwnerGroups >= n))
    p.counts[level * kWave + i] = lane < kOwnerGroups && i < n ? count : 0;
  if (blockIdx.x == 0 && lane == kOwnerGroups && p.status) *p.status = count ? HM_ERR_BAD_ID : 0;
}

struct TimeParams {
  int32_t D, G;
  int32_t U[kMaxDepth];
  double M, v;
  double fan_inter[kMaxDepth], fan_intra[kMaxDepth];   // U[i] / U[i-1] and G / U[i]
  double alpha_inter[kMaxDepth], beta_inter[kMaxDepth], alpha_intra[kMaxDepth], beta_intra[kMaxDepth];
  const int32_t *p_inter, *p_intra;
  double *times;
  int32_t *best;
};

// One wave: lane j holds entry j of each count vector; the maxima are wave reductions, the few
// fp64 operations run on lane 0 in the order the model is written (no contraction).  The vectors of
// all levels are loaded and reduced side by side, and the fan-outs U[i] / U[i-1] and G / U[d-1] come
// divided from the host: 5.5 -> 2.7 us, most of which is one trip to memory and the launch.
__global__ __launch_bounds__(kWave) void alltoall_times_kernel(TimeParams p) {
#pragma clang fp contract(off)
  const int lane = lane_id();
  int most[2 * kMaxDepth];   // p_inter of level l, then p_intra
#pragma unroll
  for (int l = 0; l < kMaxDepth; ++l) {
    most[l] = (l >= 1 && l < p.D && lane < p.U[l]) ? p.p_inter[l * kWave + lane] : 0;
    most[kMaxDepth + l] = (l < p.D && lane < p.G) ? p.p_intra[l * kWave + lane] : 0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int i = 0; i < 2 * kMaxDepth; ++i) most[i] = max(most[i], __shfl_xor(most[i], off, kWave));
  if (lane != 0) return;
  double t[kMaxDepth];
  double inter = 0.0;   // the Inter levels below the depth at hand, added up in ascending order
#pragma unroll
  for (int d = 1; d <= kMaxDepth; ++d) {
    if (d > p.D) break;
    if (d > 1) {
      const double n = p.fan_inter[d - 1] * (double)max(most[d - 1], 0) * p.M * p.v;
      inter = inter + (p.alpha_inter[d - 1] + n * p.beta_inter[d - 1]);
    }
    const double n = p.fan_intra[d - 1] * (double)max(most[kMaxDepth + d - 1], 0) * p.M * p.v;
    t[d - 1] = inter + (p.alpha_intra[d - 1] + n * p.beta_intra[d - 1]);
    p.times[d - 1] = t[d - 1];
  }
  int arg = 1;
  if (p.D > 1) {
    arg = 2;
    double least = t[1];
#pragma unroll
    for (int d = 3; d <= kMaxDepth; ++d) {
      if (d <= p.D && t[d - 1] < least) {
        least = t[d - 1];
        arg = d;
      }
    }
    if (t[0] < least) arg = 1;
  }
  *p.best = arg;
}

}  // namespace hm

extern "C" hm_status hm_group_counts(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K,
                                     int32_t E, int32_t G, int32_t depth, const int32_t *groups, int32_t *counts,
                                     int32_t *status, void *hip_stream) {
  HM_ENTRY_SCOPE;
  using namespace hm;
  if (!expert_to_rank || !groups || !counts) return HM_ERR_NULL;
  hm_status st = hm_check_tk(T, K);
  if (st != HM_OK) return st;
  if (E < 1) return HM_ERR_SHAPE;
  if (T > 0 && !topk_ids) return HM_ERR_NULL;
  if (G < 1 || G > 64 || depth < 1 || depth > kMaxDepth) return HM_ERR_TOPOLOGY;
  GroupParams p;
  for (int l = 0; l < kMaxDepth; ++l) {
    p.groups[l] = 1;
    p.per[l] = G;
  }
  for (int l = 0; l < depth; ++l) {
    if (groups[l] < 1 || groups[l] > G || G % groups[l] != 0) return HM_ERR_TOPOLOGY;
    p.groups[l] = groups[l];
    p.per[l] = G / groups[l];
  }
  p.ids = topk_ids;
  p.expert_to_rank = expert_to_rank;
  p.T = T;
  p.K = K;
  p.E = E;
  p.G = G;
  p.depth = depth;
  p.counts = counts;
  p.status = status;
  hipStream_t stream = (hipStream_t)hip_stream;
  int outputs = 0, blocks = 0;
  for (int l = 0; l < depth; ++l) {
    outputs += groups[l];
    blocks += (groups[l] + kOwnerGroups - 1) / kOwnerGroups;
  }
  // one workgroup that looks many slots up in memory is slower than several (E = 5,000, 1,024 tokens, K = 64: 32.4 us, 19.8)
  const bool alone_fits = T <= kAloneTokens && (int64_t)T * K <= 32768;
  const CountRoute route = count_route(T, K, E, outputs, blocks, false, alone_fits);
  if (route == CountRoute::kOwners || route == CountRoute::kSpread) {
    const bool spread = route == CountRoute::kSpread;
    GroupOwners o;
    for (int l = 0, first = 0; l < kMaxDepth; ++l) {
      o.first_block[l] = l < depth ? first : 0x7FFFFFFF;
      o.per_recip16[l] = (uint32_t)((65536 + p.per[l] - 1) / p.per[l]);
      first += (p.groups[l] + kOwnerGroups - 1) / kOwnerGroups;
    }
    o.tokens = spread ? spread_tokens(T, blocks) : T;
    if (spread) {
      hipLaunchKernelGGL(group_clear_kernel, dim3(1), dim3(kGroupThreads), 0, stream, p);
      if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    }
    const dim3 grid((unsigned)blocks, spread ? (unsigned)((T + o.tokens - 1) / o.tokens) : 1u);
    const int width = owner_width(K);
    const auto whole = width == 4   ? group_owner_kernel<4, false>
                       : width == 2 ? group_owner_kernel<2, false>
                                    : group_owner_kernel<1, false>;
    const auto parts = width == 4   ? group_owner_kernel<4, true>
                       : width == 2 ? group_owner_kernel<2, true>
                                    : group_owner_kernel<1, true>;
    hipLaunchKernelGGL((spread ? parts : whole), grid, dim3(kOwnerThreads), 0, stream, p, o);
    return hm_launch_status();
  }
  if (route == CountRoute::kAlone) {
    hipLaunchKernelGGL((group_count_kernel<kAloneTokens, true>), dim3(1), dim3(kAloneTokens), 0, stream, p);
    return hm_launch_status();
  }
  hipLaunchKernelGGL(group_clear_kernel, dim3(1), dim3(kGroupThreads), 0, stream, p);
  if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  int64_t all = ((int64_t)T + kGroupThreads - 1) / kGroupThreads;
  if (all > 1024) all = 1024;
  hipLaunchKernelGGL((group_count_kernel<kGroupThreads, false>), dim3((unsigned)all), dim3(kGroupThreads), 0, stream, p);
  return hm_launch_status();
}

extern "C" hm_status hm_alltoall_times(int32_t D, const int32_t *U, int32_t G, double M, double v,
                                       const int32_t *p_inter, const int32_t *p_intra, const double *alpha_inter,
                                       const double *beta_inter, const double *alpha_intra, const double *beta_intra,
                                       double *times, int32_t *best, void *hip_stream) {
  HM_ENTRY_SCOPE;
  using namespace hm;
  if (!U || !p_inter || !p_intra || !alpha_inter || !beta_inter || !alpha_intra || !beta_intra || !times || !best)
    return HM_ERR_NULL;
  if (D < 1 || D > kMaxDepth || G < 1 || G > 64 || U[0] != 1) return HM_ERR_TOPOLOGY;
  for (int i = 1; i < D; ++i)
    if (U[i] < U[i - 1] || U[i] > G || U[i] % U[i - 1] != 0 || G % U[i] != 0) return HM_ERR_TOPOLOGY;
  TimeParams p;
  p.D = D;
  p.G = G;
  p.M = M;
  p.v = v;
  for (int l = 0; l < kMaxDepth; ++l) {
    const bool in = l < D;
    p.U[l] = in ? U[l] : 1;
    p.fan_inter[l] = in && l > 0 ? (double)(U[l] / U[l - 1]) : 0.0;
    p.fan_intra[l] = in ? (double)(G / U[l]) : 0.0;
    p.alpha_inter[l] = in ? alpha_inter[l] : 0.0;
    p.beta_inter[l] = in ? beta_inter[l] : 0.0;
    p.alpha_intra[l] = in ? alpha_intra[l] : 0.0;
    p.beta_intra[l] = in ? beta_intra[l] : 0.0;
  }
  p.p_inter = p_inter;
  p.p_intra = p_intra;
  p.times = times;
  p.best = best;
  hipLaunchKernelGGL(alltoall_times_kernel, dim3(1), dim3(kWave), 0, (hipStream_t)hip_stream, p);
  return hm_launch_status();
}
