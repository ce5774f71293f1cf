// hm_expert_load: per-expert slot counts and duplicate-free per-rank / per-node token counts (the p^(1,G) and
// p^(1,U[1]) vectors of HierMoE Eq.(7)) for the expert-swap planner of Section IV.
//
// Small tables are one launch: workgroups that own a few outputs each go through all the tokens (load_owner_kernel;
// kernel trace, 8,192 x 8, 128 experts on 32 ranks: 5.2 us, 6.4 with a branch per id and a place for every four lanes).
// Larger ones: one lane per token, expert counts in an LDS histogram, rank and node counts from ballots over the
// per-token rank masks (lane g accumulates the popcount for group g), so a token is counted once per group however many
// of its experts live there; a tiny launch clears the outputs and integer atomics merge the workgroups, which keeps the
// result exact and order-independent.  The ids of a token are loaded together, while the placement is staged in LDS.
// Tried there and slower: the masks of ranks and nodes as one 64-bit word per expert in LDS and the counts by turning
// the wave's 64 x 64 bits round (6.6 us against 5.7: more code to fetch, and the ballots are not what it waits for).
#include "hm_device.h"

namespace hm {

struct LoadParams {
  const int32_t *ids;
  const int32_t *expert_to_rank;
  int32_t T, K, E, G, R, N;
  int32_t staged;   // the placement goes through LDS
  int32_t *load_expert, *load_rank, *load_node, *status;
};

constexpr int kLoadThreads = 256;
constexpr int kAloneTokens = 1024;  // = lanes of the one workgroup: one token each
constexpr int kLdsExperts = 8192;   // experts histogrammed in LDS; beyond that, global atomics

__global__ __launch_bounds__(kLoadThreads) void load_clear_kernel(LoadParams p) {
  const int i = blockIdx.x * kLoadThreads + threadIdx.x;
  if (i < p.E) p.load_expert[i] = 0;
  if (i < p.G) p.load_rank[i] = 0;
  if (i < p.N) p.load_node[i] = 0;
  if (i == 0 && p.status) *p.status = 0;
}

// ALONE: the only workgroup, for tables of more experts than can be staged; it stores the outputs instead of adding to
// cleared ones.
template <int THREADS, bool ALONE>
__global__ __launch_bounds__(THREADS) void load_count_kernel(LoadParams p) {
  __shared__ int32_t hist[kLdsExperts];
  __shared__ int8_t ranks[ALONE ? 1 : kStagedExperts];
  __shared__ int32_t rank_cnt[kWave];
  __shared__ int32_t node_cnt[kWave];
  __shared__ int32_t bad;
  const bool lds_hist = ALONE || p.E <= kLdsExperts, staged = !ALONE && p.staged;
  const int64_t stride = (int64_t)gridDim.x * THREADS;
  int64_t t = (int64_t)blockIdx.x * THREADS + threadIdx.x;
  int id[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
  if (t < p.T) load_ids(p.ids + t * p.K, p.K, 0, id);   // on their way while the tables are prepared
  if (staged)
    for (int e = threadIdx.x; e < p.E; e += THREADS) ranks[e] = rank_code(p.G, p.expert_to_rank[e]);
  if (lds_hist)
    for (int e = threadIdx.x; e < p.E; e += THREADS) hist[e] = 0;
  if (threadIdx.x < kWave) {
    rank_cnt[threadIdx.x] = 0;
    node_cnt[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();

  const int lane = lane_id();
  int my_rank_cnt = 0, my_node_cnt = 0;  // lane g: tokens of this wave's share that reach group g
  bool my_bad = false;
  // every lane of a wave runs the same number of rounds so the ballots stay convergent
  const int64_t rounds = ((int64_t)p.T + stride - 1) / stride;
  for (int64_t it = 0; it < rounds; ++it, t += stride) {
    uint64_t rm = 0;
    if (t < p.T) {
      for (int k0 = 0; k0 < p.K; k0 += 8) {
        if (it > 0 || k0 > 0) load_ids(p.ids + t * p.K, p.K, k0, id);
        auto count = [&](int slot) {
          const int g = staged ? staged_rank_of(ranks, p.E, slot) : rank_of(p.expert_to_rank, p.E, p.G, slot);
          my_bad = my_bad || g == -1;
          if (g < 0) return;
          if (lds_hist) atomicAdd(&hist[slot], 1);
          else atomicAdd(&p.load_expert[slot], 1);
          rm |= 1ull << g;
        };
        if (k0 + 8 <= p.K) {
#pragma unroll
          for (int j = 0; j < 8; ++j) count(id[j]);
        } else {   // uniform: an absent slot would cost its share of the chain all the same
#pragma unroll
          for (int j = 0; j < 7; ++j) {
            if (k0 + j >= p.K) break;
            count(id[j]);
          }
        }
      }
    }
    if (__ballot(rm != 0) == 0) continue;
    my_rank_cnt += lanes_per_group(rm, p.G, 1);
    my_node_cnt += lanes_per_group(rm, p.N, p.R);   // the ranks of a node are neighbours
  }
  if (my_bad) bad = 1;
  if (lane < p.G && my_rank_cnt) atomicAdd(&rank_cnt[lane], my_rank_cnt);
  if (lane < p.N && my_node_cnt) atomicAdd(&node_cnt[lane], my_node_cnt);
  __syncthreads();
  if (ALONE) {
    for (int e = threadIdx.x; e < p.E; e += THREADS) p.load_expert[e] = hist[e];
    if ((int)threadIdx.x < p.G) p.load_rank[threadIdx.x] = rank_cnt[threadIdx.x];
    if ((int)threadIdx.x < p.N) p.load_node[threadIdx.x] = node_cnt[threadIdx.x];
    if (threadIdx.x == 0 && p.status) *p.status = bad ? HM_ERR_BAD_ID : 0;
    return;
  }
  if (lds_hist)
    for (int e = threadIdx.x; e < p.E; e += THREADS)
      if (hist[e]) atomicAdd(&p.load_expert[e], hist[e]);
  if ((int)threadIdx.x < p.G && rank_cnt[threadIdx.x]) atomicAdd(&p.load_rank[threadIdx.x], rank_cnt[threadIdx.x]);
  if ((int)threadIdx.x < p.N && node_cnt[threadIdx.x]) atomicAdd(&p.load_node[threadIdx.x], node_cnt[threadIdx.x]);
  if (threadIdx.x == 0 && bad) flag(p.status, HM_ERR_BAD_ID);
}

// Workgroups [0, expert_blocks) own kOwnerExperts experts each, the next ones seven ranks each, the last ones seven nodes
// each; SPREAD: for a part of the tokens, added to cleared outputs.
template <int W, bool SPREAD>
__global__ __launch_bounds__(kOwnerThreads) void load_owner_kernel(LoadParams p, int expert_blocks, int rank_blocks,
                                                                   uint32_t nodes_recip16, int tokens) {
  __shared__ uint8_t table[kOwnerMaxE + 2];
  // A place per lane of a wave, so that no two lanes meet; the last row: not ours.
  __shared__ __align__(16) uint32_t cnt[kOwnerExperts + 1][kWave];
  int block = (int)blockIdx.x;
  const OwnerTokens t = owner_tokens<SPREAD>(p.ids, p.T, p.K, tokens);
  if (block < expert_blocks) {   // an id is counted whether its expert's placement is valid or not, and stored if it is
    const int e0 = block * kOwnerExperts, lane = lane_id();
    const int e = e0 + (int)(threadIdx.x >> 4);   // whose places sixteen lanes add up in the end
    bool placed = false;
    for_ids<W>(t.ids, t.T, p.K, [&] {
      if (e < p.E) placed = (unsigned)p.expert_to_rank[e] < (unsigned)p.G;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      for (int i = threadIdx.x; i < (kOwnerExperts + 1) * kWave / 4; i += kOwnerThreads) ((u32x4 *)cnt)[i] = zero;
      __syncthreads();
    }, [&](const int (&id)[2 * W], int seen, bool alive) {
      const uint32_t least = alive ? 0u : (uint32_t)kOwnerExperts;
      auto count = [&](int one, uint32_t from) {   // no branch, and no lane left out: a row per id
        const uint32_t i = min(max((uint32_t)one - (uint32_t)e0, from), (uint32_t)kOwnerExperts);
        atomicAdd(&cnt[i][lane], 1u);
      };
      if (seen == 0) {
#pragma unroll
        for (int j = 0; j < 2 * W; ++j) count(id[j], least);
      } else {
#pragma unroll
        for (int j = 0; j < 2 * W; ++j) {
          const bool again = seen < 8 ? j < seen : j >= W && j - W < seen - 8;   // uniform
          count(id[j], again ? (uint32_t)kOwnerExperts : least);
        }
      }
    }, [](bool) {});
    __syncthreads();
    const u32x4 c = *(const u32x4 *)&cnt[threadIdx.x >> 4][(threadIdx.x & 15) * 4];
    int v = (int)(c[0] + c[1] + c[2] + c[3]);
    v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);   // the lanes eight, four, two and one away in the row of sixteen
    v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, true);
    if ((threadIdx.x & 15) == 0 && e < p.E) {
      if (!SPREAD) p.load_expert[e] = placed ? v : 0;
      else if (placed && v) atomicAdd(&p.load_expert[e], v);
    }
    return;
  }
  block -= expert_blocks;
  const bool ranks = block < rank_blocks;
  const int first = (ranks ? block : block - rank_blocks) * kOwnerGroups;
  const int count = count_owned_groups<W>(t.ids, p.expert_to_rank, t.T, p.K, p.E, p.G, ranks ? 65536u : nodes_recip16, first, table);
  const int i = first + (int)threadIdx.x;
  if (threadIdx.x < kOwnerGroups && i < (ranks ? p.G : p.N)) {
    int32_t *const out = (ranks ? p.load_rank : p.load_node) + i;
    if (!SPREAD) *out = count;
    else if (count) atomicAdd(out, count);
  }
  if (block == 0 && threadIdx.x == kOwnerGroups) {
    if (SPREAD && count) flag(p.status, HM_ERR_BAD_ID);
    if (!SPREAD && p.status) *p.status = count ? HM_ERR_BAD_ID : 0;
  }
}

}  // namespace hm

extern "C" hm_status hm_expert_load(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K,
                                    int32_t E, hm_topology topo, int32_t *load_expert, int32_t *load_rank,
                                    int32_t *load_node, int32_t *status, void *hip_stream) {
  HM_ENTRY_SCOPE;
  using namespace hm;
  if (!expert_to_rank || !load_expert || !load_rank || !load_node) return HM_ERR_NULL;
  hm_status st = hm_check_tk(T, K);
  if (st != HM_OK) return st;
  if (E < 1) return HM_ERR_SHAPE;
  if (T > 0 && !topk_ids) return HM_ERR_NULL;
  st = hm_check_topology(topo);
  if (st != HM_OK) return st;
  hipStream_t stream = (hipStream_t)hip_stream;
  LoadParams p;
  p.ids = topk_ids;
  p.expert_to_rank = expert_to_rank;
  p.T = T;
  p.K = K;
  p.E = E;
  p.R = topo.ranks_per_node;
  p.G = topo.nodes * topo.ranks_per_node;
  p.N = topo.nodes;
  p.load_expert = load_expert;
  p.load_rank = load_rank;
  p.load_node = load_node;
  p.status = status;
  const int expert_blocks = (E + kOwnerExperts - 1) / kOwnerExperts, rank_blocks = (p.G + kOwnerGroups - 1) / kOwnerGroups;
  const int owner_blocks = expert_blocks + rank_blocks + (p.N + kOwnerGroups - 1) / kOwnerGroups;
  const CountRoute route = count_route(T, K, E, p.G + p.N, owner_blocks, true, T <= kAloneTokens && E <= kLdsExperts);
  const int most = E > kWave ? E : kWave;
  auto clear = [&] {
    hipLaunchKernelGGL(load_clear_kernel, dim3((most + kLoadThreads - 1) / kLoadThreads), dim3(kLoadThreads), 0, stream, p);
    return hm_launch_status();
  };
  if (route == CountRoute::kOwners || route == CountRoute::kSpread) {
    const bool spread = route == CountRoute::kSpread;
    const uint32_t nodes_recip16 = (uint32_t)((65536 + p.R - 1) / p.R);   // exact for ranks (below 64)
    const int width = owner_width(K), tokens = spread ? spread_tokens(T, owner_blocks) : T;
    if (spread && clear() != HM_OK) return HM_ERR_HIP;
    const auto whole = width == 4   ? load_owner_kernel<4, false>
                       : width == 2 ? load_owner_kernel<2, false>
                                    : load_owner_kernel<1, false>;
    const auto parts = width == 4 ? load_owner_kernel<4, true> : width == 2 ? load_owner_kernel<2, true> : load_owner_kernel<1, true>;
    const dim3 grid((unsigned)owner_blocks, spread ? (unsigned)((T + tokens - 1) / tokens) : 1u);
    hipLaunchKernelGGL((spread ? parts : whole), grid, dim3(kOwnerThreads), 0, stream, p, expert_blocks, rank_blocks, nodes_recip16,
                       tokens);
    return hm_launch_status();
  }
  if (route == CountRoute::kAlone) {
    hipLaunchKernelGGL((load_count_kernel<kAloneTokens, true>), dim3(1), dim3(kAloneTokens), 0, stream, p);
    return hm_launch_status();
  }
  int64_t blocks = ((int64_t)T + kLoadThreads - 1) / kLoadThreads;
  if (blocks > 1024) blocks = 1024;
  // Staging pays where a lane looks more slots up than it stages entries (us, staged / from memory: E = 4,096, 1,025
  // tokens, K = 1 10.1 / 7.9, K = 8 10.4 / 9.4, K = 16 11.7 / 11.4; E = 2,048, K = 16 9.9 / 10.4; 300,000 tokens, two
  // per lane, E = 2,048, K = 8 30.4 / 33.4, E = 4,096, K = 16 40.0 / 44.0).
  const int64_t lookups = blocks ? ((int64_t)T + blocks * kLoadThreads - 1) / (blocks * kLoadThreads) * K : 0;
  p.staged = E <= kStagedExperts && lookups * kLoadThreads > E;
  if (clear() != HM_OK) return HM_ERR_HIP;
  if (T == 0) return HM_OK;   // cleared outputs are the counts
  hipLaunchKernelGGL((load_count_kernel<kLoadThreads, false>), dim3((unsigned)blocks), dim3(kLoadThreads), 0, stream, p);
  return hm_launch_status();
}
