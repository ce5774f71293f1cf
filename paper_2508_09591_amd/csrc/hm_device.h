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
// tables of a few hundred KB; beyond that each should read a part of it once and add atomically to cleared outputs. A
// round of 1,024 tokens of eight ids, one token per lane, is bound by the CU's path to the caches (32 KB, 0.2 us), its
// lookups in LDS and the instructions of sixteen waves, of which there are few per id; what comes before and behind the
// rounds by its code, which runs once and cold.
constexpr int kOwnerThreads = 1024;   // = tokens of a round
constexpr int kOwnerWaves = kOwnerThreads / kWave;
constexpr int kOwnerGroups = 7;       // groups of a workgroup: the bits of a byte, but for the one that marks an error
constexpr int kOwnerRounds = 63;      // most rounds: a workgroup's sums are added in pairs of sixteen bits
constexpr int kOwnerExperts = 64;     // experts of a workgroup
constexpr int kOwnerMaxE = 4096;      // experts whose groups fit the LDS table

// Ids of a token that a lane loads together: two windows of W, 4 from four slots on, 2 for two and three, 1 (and the
// same again) for one.
static inline int owner_width(int K) { return K >= 4 ? 4 : K >= 2 ? 2 : 1; }

// count(id, seen) for every batch of up to eight ids of this lane's tokens, end() behind the last of a token.  The
// second window of a short token and the last batch of a long one overlap what was there before: `seen` (uniform) of
// the first 2 W places and, from 8 on, of the second window's, hold ids that have been counted.  Lanes without a token
// have the last one's ids; count and end are told whether they do.  The next batch is on its way meanwhile; prepare()
// runs while the first is.
template <int W, typename PREPARE, typename COUNT, typename END>
__device__ __forceinline__ void for_ids(const int32_t *__restrict__ ids, int T, int K, PREPARE prepare, COUNT count, END end) {
  const int batches = W == 4 ? (K + 7) >> 3 : 1, steps = (T + kOwnerThreads - 1) / kOwnerThreads * batches;
  const uint32_t row = (uint32_t)K * 4u, last = (uint32_t)(T - 1) * row;   // bytes; T is 64 K at most
  uint32_t at = min(__umul24(threadIdx.x, row), last);
  int t = (int)threadIdx.x, batch = 0;
  auto load = [&](int (&id)[2 * W]) {   // of the token at `at`, then on to the next batch
    const int first = K >= 8 ? min(8 * batch, K - 8) : 0, second = W == 1 ? 0 : K >= 8 ? first + 4 : K - W;
    __builtin_memcpy(&id[0], (const char *)ids + (at + 4u * (uint32_t)first), 4 * W);
    __builtin_memcpy(&id[W], (const char *)ids + (at + 4u * (uint32_t)second), 4 * W);
    if (++batch == batches) {
      batch = 0;
      at = min(at + kOwnerThreads * row, last);
    }
  };
  int counted = 0;   // batches of the present token
  auto use = [&](const int (&id)[2 * W]) {
    const bool alive = t < T;
    // places of the batch, and behind them of the second window, that an earlier one had
    const int seen = K >= 8 ? max(8 * (counted + 1) - K, 0) : 8 + 2 * W - K;
    count(id, seen, alive);
    if (++counted == batches) {
      counted = 0;
      end(alive);
      t += kOwnerThreads;
    }
  };
  int a[2 * W], b[2 * W];
  if (steps > 0) load(a);
  prepare();
#pragma unroll 1
  for (int step = 0; step < steps; step += 2) {
    if (step + 1 < steps) load(b);
    use(a);
    if (step + 1 < steps) {
      if (step + 2 < steps) load(a);
      use(b);
    }
  }
}

// Tokens with a copy in groups [first, first + 7) of ranks that r -> (r per_recip16) >> 16 puts together: returned to
// lane g of the first wave, in lane 7 the tokens with an invalid id or placement.  The table holds one bit per group an
// expert may be in, so a token's groups are the `or` of its entries; a lane keeps its counts as bytes.
template <int W>
__device__ __forceinline__ int count_owned_groups(const int32_t *__restrict__ ids, const int32_t *__restrict__ expert_to_rank,
                                                  int T, int K, int E, int G, uint32_t per_recip16, int first, uint8_t *table) {
  __shared__ u32x4 sums[kOwnerWaves];
  uint32_t low = 0, high = 0, mask = 0;
  for_ids<W>(ids, T, K, [&] {   // entry 0 is that of id -1, E + 1 of ids out of range
    for (int e = threadIdx.x; e < E + 2; e += kOwnerThreads) {
      const int g = e >= 1 && e <= E ? expert_to_rank[e - 1] : -1;
      const uint32_t in = (((uint32_t)g * per_recip16) >> 16) - (uint32_t)first;
      table[e] = (uint8_t)((unsigned)g >= (unsigned)G ? (e == 0 ? 0u : 0x80u) : in < (uint32_t)kOwnerGroups ? 1u << in : 0u);
    }
    __syncthreads();
  }, [&](const int (&id)[2 * W], int, bool) {
    uint32_t most = (uint32_t)id[0], seen = 0;
#pragma unroll
    for (int j = 1; j < 2 * W; ++j) most = max(most, (uint32_t)id[j]);
    if (__ballot(most >= (uint32_t)E) == 0) {   // two instructions an id less
#pragma unroll
      for (int j = 0; j < 2 * W; ++j) seen |= (table + 1)[(uint32_t)id[j]];
    } else {
#pragma unroll
      for (int j = 0; j < 2 * W; ++j) seen |= table[min((uint32_t)id[j] + 1u, (uint32_t)E + 1u)];
    }
    mask |= seen;
  }, [&](bool alive) {
    mask = alive ? mask : 0u;
    low += __umul24(mask & 0xFu, 0x00204081u) & 0x01010101u;   // bit i of four to byte i
    high += __umul24(mask >> 4, 0x00204081u) & 0x01010101u;
    mask = 0;
  });
  // two sums of sixteen bits in a word, over the lanes and then over the waves
  u32x4 sum;
#pragma unroll
  for (int j = 0; j < 4; ++j) sum[j] = (uint32_t)lane_scan((int)((j < 2 ? low : high) >> (8 * (j & 1)) & 0x00FF00FFu));
  if (lane_id() == kWave - 1) sums[threadIdx.x / kWave] = sum;
  __syncthreads();
  if (threadIdx.x >= kWave) return 0;
  int v = ((const int *)sums)[threadIdx.x];   // word (lane % 4) of wave (lane / 4)
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);   // the lane four away within the row of sixteen, then eight
  v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);
  v += __shfl_xor(v, 16, kWave);
  v += __shfl_xor(v, 32, kWave);
  const int g = lane_id();
  return (__shfl(v, (g >> 1 & 2) + (g & 1), kWave) >> (g & 2 ? 16 : 0)) & 0xFFFF;
}

// The tokens of a workgroup: all, or, where a larger table is spread over workgroups that add to cleared outputs,
// `share` of them from blockIdx.y on.
struct OwnerTokens {
  const int32_t *ids;
  int T;
};
template <bool SPREAD>
__device__ __forceinline__ OwnerTokens owner_tokens(const int32_t *ids, int T, int K, int share) {
  if (!SPREAD) return {ids, T};
  const int64_t from = (int64_t)blockIdx.y * share;
  return {ids + from * K, (int)min((int64_t)share, T - from)};
}
// Tokens of a workgroup: whole rounds, as few as fill the chip once.
static inline int spread_tokens(int64_t T, int64_t blocks) {
  const int64_t rounds = (T + kOwnerThreads - 1) / kOwnerThreads, each = (rounds * blocks + 255) / 256;
  return (int)(each < 1 ? 1 : each > kOwnerRounds ? kOwnerRounds : each) * kOwnerThreads;
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

// Which kernel takes the counts of a table (hm_expert_load, hm_group_counts); outputs: the groups of all levels, or
// ranks and nodes; blocks: the workgroups that own them.  All figures: graphs of ten calls; lines through 4,000 shapes
// of 16 to 65,536 and 2,500 of 512 to a million tokens, one to 64 ids, 2 to 2,048 experts, even and Zipf ids, dropped
// slots.
//  * kOwners, one launch, for few rounds of 1,024 tokens.  A round costs 0.2 us with one id per token, 0.25 with two or
//    three, 0.45 with four to seven (two loads that overlap), 0.36 with eight, as much per eight of more, and twice
//    that where a token's row is 100 bytes or more, whose lines no two lanes share.  Loads of 8,192 x 8, 128 experts on
//    32 ranks 5.9 us (kAdded 7.7), group counts with four levels of 32 ranks 6.3 (8.1).
//  * kSpread: the owners' work on a part of the tokens each, as few rounds as fill the chip once, added to outputs that
//    a launch before clears: where that is a us faster, as a launch costs the host more, and for up to sixteen ids and
//    12 us of rounds: beyond, every table is read too often.  Against kAdded 0.74 times as long up to 64 rounds, 0.5 to
//    0.7 beyond (16,384 x 8, four levels of 32 ranks 7.4 -> 5.6), but 1.3 with 24 ids of 250,000 tokens (group counts
//    21 -> 35).
//  * kAdded otherwise, unless the owners, which read a long row better than the lanes of kAdded, are faster for one or
//    two rounds.
//  * kAlone, one workgroup, as far as it goes, where the owners' table has no room, and so none of kStagedExperts
//    either; 1.3 times as slow as owners where it has.
// Of 3,500 shapes drawn anew, up to 260,000 tokens, 11 are more than 3 % slower than before there were windows and
// spreading: nine of 64 ids, eight of a few hundred tokens, 3 to 7 % (loads of 469 x 64, 74 experts 6.9 -> 7.3; groups
// of 673 x 64 8.2 -> 8.6; loads of 60,530 x 64 21.4 -> 22.1), loads of 193,548 x 31, 1,690 experts, 27.8 -> 29.3, and
// loads of 90,003 x 10, 874 experts by Zipf on 64 ranks, 17.1 -> 20.0.
static_assert(hm::kOwnerMaxE >= hm::kStagedExperts, "kAlone looks placements up in memory");
enum class CountRoute { kAlone, kOwners, kSpread, kAdded };
static inline CountRoute count_route(int64_t T, int64_t K, int64_t E, int64_t outputs, int64_t blocks, bool loads, bool alone_fits) {
  if (E > hm::kOwnerMaxE) return alone_fits ? CountRoute::kAlone : CountRoute::kAdded;
  const int64_t rounds = (T + hm::kOwnerThreads - 1) / hm::kOwnerThreads, batches = (K + 7) / 8;
  const int64_t step = K == 1 ? 20 : K <= 3 ? 25 : K < 8 ? 45 : K == 8 ? 36 : K <= 24 ? 43 : 85;   // hundredths of a us, as all below
  const int64_t owners = 295 + step * batches * rounds + E / 50 + outputs / 5;
  const int64_t share = step * batches * (hm::spread_tokens(T, blocks) / hm::kOwnerThreads);
  if (K <= 16 && share <= 1200)
    return rounds <= hm::kOwnerRounds && owners <= 585 + share * 11 / 10 ? CountRoute::kOwners : CountRoute::kSpread;
  const int64_t tokens = T < 65536 ? T : 65536;
  const int64_t added = loads ? 520 + 15 * K + outputs * 24 / 10 + E * 8 / 100 + tokens * 56 / 10000
                              : 525 + 9 * K + outputs * 35 / 10 + E * 4 / 100 + tokens * 40 / 10000;
  return rounds <= hm::kOwnerRounds && owners <= added ? CountRoute::kOwners : CountRoute::kAdded;
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
