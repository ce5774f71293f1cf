// Device-side helpers shared by the gfx950 kernels of libhiermoe (wave64 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hiermoe.h"

namespace hm {

constexpr int kWave = 64;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_align2 __attribute__((aligned(2)));   // the same at the alignment of a bf16 / fp32 element
typedef u32x4 u32x4_align4 __attribute__((aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Sticky error word: codes are negative and the most negative one wins, so the result does not
// depend on the order in which waves report.
__device__ __forceinline__ void flag(int32_t *status, int32_t code) {
  if (status) atomicMin(status, code);
}

// Rank of an expert id; -1 when the id or the placement entry is out of range (an error), -2 for
// the id -1, the marker of a slot the router dropped (skipped everywhere, not an error).
__device__ __forceinline__ int rank_of(const int32_t *__restrict__ expert_to_rank, int E, int G, int id) {
  if (id == -1) return -2;
  if ((unsigned)id >= (unsigned)E) return -1;
  const int g = expert_to_rank[id];
  return ((unsigned)g >= (unsigned)G) ? -1 : g;
}

// The same with the table staged in LDS as rank_code() wrote it, for E up to kStagedExperts; a lane that
// looks up several ids then waits for LDS, not for a second trip to memory per id.
constexpr int kStagedExperts = 4096;
__device__ __forceinline__ int8_t rank_code(int G, int g) { return (unsigned)g >= (unsigned)G ? -1 : (int8_t)g; }
__device__ __forceinline__ int staged_rank_of(const int8_t *ranks, int E, int id) {
  if (id == -1) return -2;
  return (unsigned)id >= (unsigned)E ? -1 : ranks[id];
}

// Eight ids of a token from k0 on (-1, the marker of a dropped slot, past its end), loaded together.
__device__ __forceinline__ void load_ids(const int32_t *__restrict__ tok, int K, int k0, int (&id)[8]) {
  if (k0 + 8 <= K) {
    __builtin_memcpy(id, tok + k0, sizeof(id));
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) id[j] = k0 + j < K ? tok[k0 + j] : -1;
  }
}

// How many of the wave's lanes have a bit of group j of `mask` set, in lane j < n: the mask is cut into n
// groups of `per` bits.  Eight groups at a time: a ballot and its population count are a chain
// between the vector and the scalar unit that one wave alone does not hide.
__device__ __forceinline__ int lanes_per_group(uint64_t mask, int n, int per) {
  const int lane = lane_id();
  const uint64_t field = per >= 64 ? ~0ull : (1ull << per) - 1ull;
  int mine = 0;
  for (int j0 = 0; j0 < n; j0 += 8) {
    int c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = __popcll(__ballot((mask & (field << min((j0 + i) * per, 63))) != 0));
#pragma unroll
    for (int i = 0; i < 8; ++i) mine = lane == j0 + i ? c[i] : mine;
  }
  return lane < n ? mine : 0;
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ int lane_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);    // from the lane one below, within rows of sixteen
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // lane 15 of a row to the next one, rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // lane 31 to rows 2 and 3
  return v;
}

// ---- counts by owners ----------------------------------------------------------------------------------
// Counts of a routing table in one launch without cleared outputs: a workgroup owns a few outputs (seven groups, or
// some experts), goes through all the tokens and stores its counts.  The workgroups read the same table, so this is for
// tables of a few hundred KB; beyond that each should read a part of it once and add atomically to cleared outputs.
// A round of 1,024 tokens, one per lane, is bound by issuing its instructions (sixteen waves on a CU, four cycles
// each: 0.4 us for eight ids), so there are few per id.  More rounds in flight, or four ids per lane, gained nothing.
constexpr int kOwnerThreads = 1024;   // = tokens of a round
constexpr int kOwnerGroups = 7;       // groups of a workgroup: the bits of a byte, but for the one that marks an error
constexpr int kOwnerExperts = 64;     // experts of a workgroup ...
constexpr int kOwnerCopies = 4;       // ... each counted in four places, so that fewer lanes meet at one
constexpr int kOwnerMaxE = 4096;      // experts whose groups fit the LDS table

// count(id) for every id of this lane's tokens, eight lookups side by side, end() after the last of a token.  The next
// eight are on their way meanwhile; prepare() runs while the first are.  Lanes without a token count ids of -1.
template <typename PREPARE, typename COUNT, typename END>
__device__ __forceinline__ void for_ids(const int32_t *__restrict__ ids, int T, int K, PREPARE prepare, COUNT count, END end) {
  int t = (int)threadIdx.x, k0 = 0;
  const int32_t *at = ids + (int64_t)t * K;
  const int steps = (T + kOwnerThreads - 1) / kOwnerThreads * ((K + 7) >> 3);
  int id[8], next[8];
  auto load = [&](int n) {   // n ids of the token are left
#pragma unroll
    for (int j = 0; j < 8; ++j) next[j] = -1;
    if (t < T) {
      if (n >= 8) {
        __builtin_memcpy(next, at, sizeof(next));
      } else {
#pragma unroll
        for (int j = 0; j < 7; ++j)
          if (j < n) next[j] = at[j];
      }
    }
  };
#pragma unroll 1
  for (int step = -1; step < steps; ++step) {
#pragma unroll
    for (int j = 0; j < 8; ++j) id[j] = step < 0 ? -1 : next[j];
    const int n = K - k0;
    if (step >= 0) {
      at += n > 8 ? 8 : (int64_t)kOwnerThreads * K - k0;
      t += n > 8 ? 0 : kOwnerThreads;
      k0 = n > 8 ? k0 + 8 : 0;
    }
    load(K - k0);
    if (step < 0) {
      prepare();
      continue;
    }
    if (n >= 8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) count(id[j]);
    } else {   // an absent id would cost as much as any other
#pragma unroll
      for (int j = 0; j < 7; ++j)
        if (j < n) count(id[j]);
    }
    if (n <= 8) end();
  }
}

// Tokens with a copy in groups [first, first + 7) of `per` ranks each -> cnt[0 .. 7) of the workgroup's LDS, valid after the
// call for every lane; returns whether any id or placement is invalid.  The table holds one bit per group an expert
// may be in, so a token's groups are the `or` of its entries; a lane keeps its counts as bytes (at most 255 rounds).
__device__ __forceinline__ bool count_owned_groups(const int32_t *__restrict__ ids, const int32_t *__restrict__ expert_to_rank, int T, int K,
                                                   int E, int G, int per, int first, uint8_t *table, int32_t *cnt) {
  const uint32_t per_recip16 = (65536u + (uint32_t)per - 1u) / (uint32_t)per;   // exact for ranks (below 64)
  uint32_t low = 0, high = 0, mask = 0;
  for_ids(ids, T, K, [&] {   // entry 0 is that of id -1, E + 1 of ids out of range
    for (int e = threadIdx.x; e < E + 2; e += kOwnerThreads) {
      const int g = e >= 1 && e <= E ? expert_to_rank[e - 1] : -1;
      const uint32_t in = (((uint32_t)g * per_recip16) >> 16) - (uint32_t)first;
      table[e] = (uint8_t)((unsigned)g >= (unsigned)G ? (e == 0 ? 0u : 0x80u) : in < (uint32_t)kOwnerGroups ? 1u << in : 0u);
    }
    if (threadIdx.x < 8) cnt[threadIdx.x] = 0;
    __syncthreads();
  }, [&](int id) { mask |= table[min((uint32_t)id + 1u, (uint32_t)E + 1u)]; }, [&] {
    low += (mask & 0xFu) * 0x00204081u & 0x01010101u;   // bit i of four to byte i
    high += (mask >> 4) * 0x00204081u & 0x01010101u;
    mask = 0;
  });
  // two sums of sixteen bits in a word, over the lanes and then over the waves; the eighth counts tokens with an error
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int v = lane_scan((int)((j < 2 ? low : high) >> (8 * (j & 1)) & 0x00FF00FFu));
    if (lane_id() == kWave - 1) {
      atomicAdd(&cnt[4 * (j >> 1) + (j & 1)], v & 0xFFFF);
      atomicAdd(&cnt[4 * (j >> 1) + (j & 1) + 2], v >> 16);
    }
  }
  __syncthreads();
  return cnt[kOwnerGroups] != 0;
}

// Value held by lane `src` (src must be wave-uniform).
__device__ __forceinline__ int read_lane(int v, int src) { return __builtin_amdgcn_readlane(v, src); }
__device__ __forceinline__ float read_lane(float v, int src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
}

// bf16 pair packed in one 32-bit word -> two floats (low half first).
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }

// float -> bf16 encoding, round to nearest even; NaN maps to the quiet NaN 0x7FC0.
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16(lo) | (f32_to_bf16(hi) << 16);
}

}  // namespace hm

// Which kernel takes the counts of a table (hm_expert_load, hm_group_counts); outputs: the groups of all levels, or ranks and nodes.
//  * kOwners where the rounds of 1,024 tokens cost less than the clearing launch, the gap behind it and the atomics.  A round costs
//    0.38 us per eight ids (0.47 if there are more) and for the ids that are left, which take a load of a word each, 0.45 up to
//    three, 0.8 for four and five, 1.0 and 1.35 for six and seven, the more the longer the tokens; what it saves is 2 us, 0.036 per output (the
//    ballots of the other kernels), 0.1 per id of a load and 0.06 per id beyond eight.  Graphs of ten calls, us, clear + count
//    -> owners: group counts of 8,192 x 8 with four levels of 32 ranks 7.9 -> 7.1, with one of 16 6.5 -> 6.9 (6,144 tokens: 6.4 -> 6.1);
//    4,096 x 2 6.1 -> 5.6, x 4 6.1 -> 7.0, x 7 6.2 -> 8.6 (2,048 x 7 with four levels 7.7 -> 6.1); loads of 8,192 x 8 on 32 ranks 7.7 -> 6.7,
//    4,096 x 7 7.5 -> 8.7, x 12 8.3 -> 8.7, 2,048 x 31 10.5 -> 11.8.  Few experts make many lanes meet at one count (E = 32, 16
//    ranks, 8,192 x 8: 7.1 -> 7.5).  And a launch less takes 2.4 us off the host.
//  * kAlone, one workgroup, for a few tokens with few outputs (and, for loads, ids), as an owner works out an entry of a table per
//    expert: 64 tokens, groups of 8 ranks, E = 128 3.85, owners 4.05, E = 2,048 4.05, 4.5; loads of one id, 8 ranks 3.75, 4.1; but
//    four levels of 32 ranks 5.6, 4.4.  And, as far as it goes, where the owners' table has no room.
enum class CountRoute { kAlone, kOwners, kAdded };
static inline CountRoute count_route(int64_t T, int64_t K, int64_t E, int64_t outputs, bool loads, bool alone_fits) {
  const int64_t few = E / 128 + (!loads ? 8 : K == 1 ? 20 : K <= 3 ? 10 : -E / 128);
  if (alone_fits && outputs <= few && (T <= 256 || (T <= 512 && K <= 2 && outputs <= 10 + E / 128)) && K <= 8) return CountRoute::kAlone;
  static const int left[8] = {0, 45, 45, 45, 80, 80, 100, 135}, longer[4] = {4, 5, 6, 9};   // hundredths of a us, quarters
  const int64_t rounds = (T + hm::kOwnerThreads - 1) / hm::kOwnerThreads, steps = rounds * ((K + 7) / 8);
  const int64_t round = K / 8 * (K > 8 || (loads && E < 64) ? 47 : 38) + left[K % 8] * longer[K < 32 ? K / 8 : 3] / 4;
  const int64_t saved = 200 + outputs * 36 / 10 + (loads ? 10 * K : 0) + (K > 8 ? 6 * (K - 8) : 0);
  const bool pays = steps <= (K < 8 || E < 32 ? 4 : 8) && (rounds <= 1 || rounds * round <= saved);
  if (pays && E <= hm::kOwnerMaxE) return CountRoute::kOwners;
  return alone_fits ? CountRoute::kAlone : CountRoute::kAdded;
}

// Host-side argument checks shared by the entry points.
static inline hm_status hm_check_topology(hm_topology topo) {
  if (topo.nodes < 1 || topo.ranks_per_node < 1) return HM_ERR_TOPOLOGY;
  if (topo.nodes > 32 || topo.ranks_per_node > 64) return HM_ERR_TOPOLOGY;
  if ((int64_t)topo.nodes * topo.ranks_per_node > 64) return HM_ERR_TOPOLOGY;
  return HM_OK;
}
static inline hm_status hm_check_tk(int32_t T, int32_t K) {
  if (T < 0 || K < 1 || K > 64) return HM_ERR_SHAPE;
  if ((int64_t)T * K > 2147483647LL) return HM_ERR_SHAPE;
  return HM_OK;
}
// Launch errors.  HIP keeps the last error of a thread until somebody reads it, so an error the
// host program left behind before calling into this library must not be reported as a failed
// launch of ours (nor cleared: it is the host program's to find).  Every entry point notes what
// was pending when it was entered; a launch counts as failed only if a new error appears.
static thread_local hipError_t hm_pending_at_entry = hipSuccess;
struct hm_entry_scope {
  hm_entry_scope() { hm_pending_at_entry = hipPeekAtLastError(); }
};
#define HM_ENTRY_SCOPE const hm_entry_scope hm_entry_scope_here
static inline hm_status hm_launch_status() {
  const hipError_t now = hipPeekAtLastError();
  if (now == hipSuccess || now == hm_pending_at_entry) return HM_OK;
  (void)hipGetLastError();   // ours: reported through the return code, not left for the next caller
  return HM_ERR_HIP;
}
