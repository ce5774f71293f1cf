// hm_plan: routing -> deduplicated, stable per-destination send lists (HierMoE Eq.(7)).
//
// One lane owns one routing slot s = t*K + k; a wave owns 64 consecutive slots, a workgroup 1024.
// Rows of a destination are numbered in ascending slot order, so a lane's row is
//     dest_offset[d] + (kept slots of d in earlier workgroups) + (in earlier waves of this
//     workgroup) + (in lower lanes of this wave),
// and the last term is a count of bits below the lane's own in a 64-bit word per (wave, destination).  No order
// of atomics decides positions, so the plan is deterministic and stable.  A workgroup first stages the
// destinations of its tokens (its 1024 slots and the rest of its first and last token) in LDS: each expert id is
// looked up once and all "same destination as an earlier / later slot of my token" questions become
// comparisons of eight bytes.
//
// Every workgroup needs the counts of all the others (the destination totals give dest_offset),
// so the plan has a grid-wide dependency in the middle.  A plan of one workgroup has none
// (plan_alone_kernel: 128 tokens of 8 slots 5.2 us by kernel trace).  Otherwise there are two ways through it:
//   * plans of at most 256 workgroups (262,144 slots) run as ONE launch, plan_fused_kernel: the
//     workgroups publish their counts, wait for one another's and go on to write the maps from
//     what they staged.  At these sizes the work is a few microseconds and a second launch (its
//     gap, and staging everything again) cost more than the kernels themselves.  All workgroups
//     are resident together (the launcher checks the device's capacity), the counts carry a value
//     unique to the launch, so the caller's workspace needs no initialisation, and every wait is
//     bounded: a wave that gives up flags HM_ERR_HIP and exits.
//   * larger plans take separate launches: plan_count_kernel (per-workgroup counts ->
//     workspace), plan_scan_kernel once the matrix has kPlanScanMinEntries entries (one
//     workgroup per destination turns it into exclusive prefixes plus a row of totals; below
//     that every workgroup re-reads the small matrix itself), and plan_write_kernel: the body of
//     the one-launch kernel without its grid-wide wait (the counts are complete when it starts).
//     Linear in the number of slots at any size.
#include "hm_device.h"

#include <unistd.h>

#include <atomic>
#include <chrono>
#include <mutex>

namespace hm {

constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kPlanHalo = 63;                              // K - 1 <= 63
constexpr int64_t kPlanScanMinEntries = 16384;             // count-matrix entries from which the scan launch pays
constexpr int kPlanFusedMaxBlocks = 256;                   // largest plan (in workgroups) the one-launch kernel takes
constexpr int kPlanSpinLimit = 1 << 18;                    // polls of the grid barrier before a wave gives up
constexpr int kPlanStagedExperts = 4096;                   // one-launch kernel: largest expert table staged in LDS

struct PlanParams {
  const int32_t *ids;
  const float *weights;
  const int32_t *expert_to_rank;
  const int32_t *dest_map;  // non-null: destinations come from this table (hm_plan_mapped)
  int32_t T, K, E, G, R, N, Dn, level;   // N = G / R nodes
  int32_t nslots, nblocks;
  uint64_t k_recip;      // ceil(2^64 / K), 0 for K = 1
  uint32_t k_recip22;    // ceil(2^22 / K): exact for numerators below 1024 + 128, K <= 64
  uint32_t r_recip16;    // ceil(2^16 / R): exact for ranks (below 64)
  int32_t scanned;  // counts holds exclusive prefixes over workgroups and the totals in row nblocks
  int64_t row_capacity;
  int32_t *counts;  // workspace [nblocks + 1][Dn]
  int32_t *dest_count, *dest_offset, *row_token, *slot_row;
  uint8_t *slot_keep;
  float *row_weight;
  uint64_t *rank_mask;
  uint32_t *node_mask;
  int32_t *status;
  int32_t *load_expert, *load_rank, *load_node;  // optional: the counts of hm_expert_load, fused
};

// Words that another workgroup of the same launch reads or writes are accessed with device-scope
// atomic loads and stores (the workgroups sit on different dies with caches of their own).
__device__ __forceinline__ void st_device(int32_t *a, int32_t v) {
  __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_device(const uint64_t *a) {
  return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_device(uint64_t *a, uint64_t v) {
  __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The calling wave's earlier device-scope stores have been acknowledged when this returns.
__device__ __forceinline__ void wait_for_own_stores() { __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- the slots of a workgroup --------------------------------------------------------------------
// The destinations of the workgroup's tokens lie in LDS as bytes, token by token, each token padded to whole
// 8-byte words (kNoCopy and above: no copy).  Which other slots of its token share a lane's destination is then one
// comparison of eight bytes at a time instead of a loop over the slots.
//
// What a plan kernel spends its time on is neither memory nor arithmetic but the instruction stream: a workgroup
// runs its code once, from a cold instruction cache, at about 0.5 ns per byte (a probe of straight-line code: 7 KB 4.2
// us, 28 KB 14.9), and sixteen waves issue each instruction in turn.  So the steps below are chosen for few
// instructions, and nothing is unrolled or expanded twice that need not be:
//   * an expert's rank and node come from one 16-bit LDS entry;
//   * the slots of a wave with the same destination are a 64-bit LDS word per (wave, destination), one `or` per
//     slot, instead of a ballot per bit of the destination; its bits below a lane are the lane's position, its
//     number of bits the wave's count, kept as a byte, so that the sums over sixteen waves are a few byte sums;
//   * masks and duplicate-free loads are worked out while the workgroups wait for one another, and of the loads
//     only those that are not the rows' own counts.  (Atomic `or`s and adds in LDS for them, by which eight and more
//     lanes meet at one word, took 0.2 to 0.4 us each, a loop over the ranks with a ballot each 60 ns a turn.)
// Kernel trace, before -> after, us: 1,024 x 2 slots 7.9 -> 5.8, 128 x 8 6.2 -> 5.2, 8,192 x 8 at rank level 8.1 -> 6.8, at node
// level 9.1 -> 6.8, 4,097 x 6 without dedup 8.2 -> 6.4, 25,600 x 8 through a hop table 12.5 -> 10.3.
struct Tokens {
  int first_slot, first_token, tokens, words;   // of the workgroup; 8-byte words per token
};
__device__ __forceinline__ int token_of_slot(const PlanParams &p, int s) {
  return p.k_recip ? (int)__umul64hi((uint64_t)(unsigned)s, p.k_recip) : s;
}
__device__ __forceinline__ int node_of(const PlanParams &p, int rank) { return (int)(((uint32_t)rank * p.r_recip16) >> 16); }
__device__ __forceinline__ Tokens tokens_of_block(const PlanParams &p) {
  Tokens k;
  k.first_slot = (int)blockIdx.x * kPlanThreads;
  k.first_token = token_of_slot(p, k.first_slot);
  const int slots = min(kPlanThreads, p.nslots - k.first_slot);   // none in an empty plan
  k.tokens = slots < 1 ? 0 : token_of_slot(p, k.first_slot + slots - 1) - k.first_token + 1;
  k.words = (p.K + 7) >> 3;
  return k;
}
// Token (counted from the workgroup's first) and place in it of a slot of the workgroup's tokens.
__device__ __forceinline__ int token_of(const PlanParams &p, const Tokens &k, int s, int &place) {
  const unsigned q = (unsigned)(s - k.first_token * p.K);
  const int t = (int)((q * p.k_recip22) >> 22);
  place = (int)q - t * p.K;
  return t;
}
// 0x80 in every byte of w that equals the byte repeated in `same`.
__device__ __forceinline__ uint64_t equal_bytes(uint64_t w, uint64_t same) {
  const uint64_t x = w ^ same, low = 0x7F7F7F7F7F7F7F7Full;
  return ~(((x & low) + low) | x | low);
}
__device__ __forceinline__ uint64_t repeated(int byte) {
  const uint32_t four = (uint32_t)byte * 0x01010101u;
  return (uint64_t)four << 32 | four;
}

// What an expert id stands for: the rank (hop tables: the destination) in the low byte, its node in the next one.
// 0xFF in both is an error, 0xFE in both no copy: an id of -1 (a slot the router dropped) or a hop table's -1.
constexpr uint32_t kBadEntry = 0xFFFFu, kNoCopy = 0xFEFEu;
__device__ __forceinline__ uint32_t table_entry(const PlanParams &p, int e) {
  const int g = p.dest_map ? p.dest_map[e] : p.expert_to_rank[e];
  const uint32_t entry = (uint32_t)g | (uint32_t)node_of(p, g) << 8;   // hop tables: ranks_per_node is 1
  return (unsigned)g < (unsigned)p.G ? entry : p.dest_map && g == -1 ? kNoCopy : kBadEntry;
}
// staged: the table in LDS, with an entry for ids out of range behind the last expert's.
__device__ __forceinline__ uint32_t entry_of(const PlanParams &p, const uint16_t *staged, int id) {
  uint32_t entry;
  if (staged) entry = staged[min((unsigned)id, (unsigned)p.E)];
  else entry = (unsigned)id < (unsigned)p.E ? table_entry(p, id) : kBadEntry;
  return id == -1 ? kNoCopy : entry;
}

// Bytes of a workgroup's tokens: most with K = 1, a word per slot.
constexpr int kPlanTokenWords = kPlanThreads + 2;

// A halo slot of this lane, if it has one: the slots of the first token before the workgroup's, those of
// the last token behind it.
__device__ __forceinline__ int halo_slot(const PlanParams &p, const Tokens &k) {
  const int before = k.first_slot - k.first_token * p.K;               // < K
  const int i = (int)threadIdx.x;
  if (i < before) return k.first_token * p.K + i;
  const int64_t s = (int64_t)k.first_slot + kPlanThreads + (i - before);
  return s < (int64_t)(k.first_token + k.tokens) * p.K ? (int)s : -1;
}

struct PlanShared {
  alignas(16) uint32_t wave_cnt[kWave][kPlanWaves / 4];   // per (destination, wave): rows it owns, as bytes
  uint64_t dest_bytes[kPlanTokenWords];
  uint64_t other_bytes[kPlanTokenWords];             // ranks where the destinations are nodes, nodes where they are ranks
  float weight[kPlanThreads + kPlanHalo];
  unsigned long long same_dest[kPlanWaves][kWave];   // per (wave, destination): the lanes that own a row there
  int32_t rank_cnt[kWave], node_cnt[kWave];          // the workgroup's tokens per rank and node
  int32_t all_tot[kWave], all_pre[kWave];            // per destination: rows of the plan, of the workgroups before
  int32_t gave_up;
};

// One lane's slot.
struct Slot {
  int s, id, tok, place, dest;   // dest: kNoCopy's or kBadEntry's byte if there is none
  uint32_t entry;
  float w;
  int other;                     // the node if dest is a rank, the rank if it is a node
  bool live, has_dest, first, keep;   // first slot of its token with this destination; owner of a row
  int pos;                       // among the rows of the wave with the same destination
};

// Whether no slot of the token before `place` has this byte.
__device__ __forceinline__ bool first_in_token(const uint64_t *bytes, const Tokens &k, int tok, int place, int byte) {
  const uint64_t same = repeated(byte);
  bool first = true;
#pragma unroll 1
  for (int wd = 0; wd < k.words; ++wd) {
    const int at = place - 8 * wd;   // counted from this word's first
    const uint64_t not_before = at <= 0 ? ~0ull : at >= 8 ? 0ull : ~0ull << (8 * at);
    first = first && (equal_bytes(bytes[tok * k.words + wd], same) & ~not_before) == 0;
  }
  return first;
}

// The bits of eight bytes of a token, by each of eight neighbouring lanes (words from k.words on: none), then of them all.
template <typename MASK>
__device__ __forceinline__ MASK mask_of_words(const uint64_t *bytes, const Tokens &k, int tok, int wd) {
  const uint64_t w = wd < k.words ? bytes[tok * k.words + wd] : ~0ull;
  MASK mask = 0;
#pragma unroll 1
  for (int j = 0; j < 64; j += 8) {
    const uint32_t b = (uint32_t)(w >> j) & 0xFFu;
    mask |= b < kWave ? (MASK)1 << b : (MASK)0;
  }
#pragma unroll 1
  for (int off = 1; off < 8; off <<= 1) mask |= __shfl_xor(mask, off, kWave);
  return mask;
}

// The bits of a token's bytes.
template <typename MASK>
__device__ __forceinline__ MASK mask_of_token(const uint64_t *bytes, const Tokens &k, int K, int tok) {
  MASK mask = 0;
#pragma unroll 1
  for (int wd = 0; wd < k.words; ++wd) {
    const uint64_t w = bytes[tok * k.words + wd];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (8 * wd + j >= K) break;
      const uint32_t b = (uint32_t)(w >> (8 * j)) & 0xFFu;
      mask |= b < kWave ? (MASK)1 << b : (MASK)0;
    }
  }
  return mask;
}

// Everything up to the wave's counts, in two steps with the barriers between: COUNT_ONLY leaves out what only the
// maps need.  `hist` and `table` are LDS behind PlanShared, null if not used.  THREADS: lanes of the workgroup, kPlanThreads
// unless it is the only one.
template <bool COUNT_ONLY, int THREADS>
__device__ __forceinline__ Slot plan_slots(const PlanParams &p, PlanShared &sh, const Tokens &k, int32_t *hist, uint16_t *table,
                                           bool own_status) {
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), tid = (int)threadIdx.x;
  const bool loads = !COUNT_ONLY && p.load_expert != nullptr, tokens = loads || (!COUNT_ONLY && (p.rank_mask || p.node_mask));
  Slot me;
  // everything that comes from memory, in one round: this lane's slot, its halo slot, the table
  me.s = k.first_slot + tid;
  me.live = me.s < p.nslots;
  // One workgroup has all of its tokens.  There are at most 2 (K - 1) = 126 halo slots, so only the first two waves
  // look for one (all sixteen: 200,000 x 3 slots 29.6 -> 31.9 us, 52,429 x 5 at node level 13.7 -> 14.5).
  const bool halo = wv < 2 && p.nblocks > 1 && (kPlanThreads % (unsigned)p.K) != 0;
  const int s2 = halo ? halo_slot(p, k) : -1;
  int id2 = -1;
  float w2 = 0.0f;
  me.id = -1;
  me.w = 0.0f;
  if (me.live) {
    me.id = p.ids[me.s];
    if (!COUNT_ONLY) me.w = p.weights[me.s];
  }
  if (halo && s2 >= 0) {
    id2 = p.ids[s2];
    if (!COUNT_ONLY) w2 = p.weights[s2];
  }
  if (own_status && tid == 0) st_device(p.status, 0);
  if (table)
    for (int e = tid; e <= p.E; e += THREADS) table[e] = (uint16_t)(e < p.E ? table_entry(p, e) : kBadEntry);
  if (loads && hist)
    for (int e = tid; e < p.E; e += THREADS) hist[e] = 0;
  for (int i = tid; i < k.tokens * k.words; i += THREADS) sh.dest_bytes[i] = sh.other_bytes[i] = ~0ull;
  sh.same_dest[wv][lane] = 0;
  if (tid < kWave) {
    sh.rank_cnt[tid] = sh.node_cnt[tid] = sh.all_tot[tid] = sh.all_pre[tid] = 0;
    sh.gave_up = 0;
  }
  if (own_status) wait_for_own_stores();   // status and cleared loads: out before anything adds to them
  __syncthreads();

  // ranks and nodes of the workgroup's tokens into LDS: this lane's slot, then its halo slot
  const int shift = p.level == HM_DEDUP_NODE && !p.dest_map ? 8 : 0;
  me.tok = token_of(p, k, me.s, me.place);
  me.entry = entry_of(p, table, me.id);
  me.dest = (int)(me.entry >> shift & 0xFFu);
  me.has_dest = me.entry < (kNoCopy & 0xFF00u);
  if (!COUNT_ONLY) sh.weight[tid] = me.w;
  if (loads && me.has_dest && hist) atomicAdd(&hist[me.id], 1);
  {
    int tok = me.tok, place = me.place, dest = me.dest;
    uint32_t entry = me.entry;
    bool in = me.live;
#pragma unroll 1
    for (int pass = 0;; ++pass) {
      if (in && entry < (kNoCopy & 0xFF00u)) {
        const int at = tok * k.words * 8 + place;
        ((uint8_t *)sh.dest_bytes)[at] = (uint8_t)dest;
        if (tokens) ((uint8_t *)sh.other_bytes)[at] = (uint8_t)(entry >> (8 - shift));
      }
      if (!halo || pass) break;
      in = s2 >= 0;
      tok = token_of(p, k, in ? s2 : me.s, place);
      entry = entry_of(p, table, id2);
      dest = (int)(entry >> shift & 0xFFu);
      if (!COUNT_ONLY && in && s2 > me.s) sh.weight[s2 - k.first_slot] = w2;   // behind the workgroup's own
    }
  }
  __syncthreads();

  // A slot owns its (token, destination) row at level none always, else iff no earlier slot of the token
  // has the same destination: the OR over a group's experts in Eq.(7) leaves one copy per group, and
  // the lowest k keeps it.
  me.other = (int)(me.entry >> (8 - shift) & 0xFFu);
  me.first = me.has_dest;
  if (p.level != HM_DEDUP_NONE || loads) me.first = me.first && first_in_token(sh.dest_bytes, k, me.tok, me.place, me.dest);
  me.keep = p.level != HM_DEDUP_NONE ? me.first : me.has_dest;
  // LDS operations of one wave are carried out in order: no barrier up to the counts
  if (me.keep) atomicOr(&sh.same_dest[wv][me.dest], 1ull << lane);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // for the compiler: no instruction
  const uint64_t peers = sh.same_dest[wv][me.dest & (kWave - 1)];
  me.pos = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
  ((uint8_t *)sh.wave_cnt)[lane * kPlanWaves + wv] = (uint8_t)__popcll(sh.same_dest[wv][lane]);
  __syncthreads();
  return me;
}

// Rows that the waves of the workgroup own at destination `lane`: all of them, and those of the waves before wv.
__device__ __forceinline__ int byte_sum(uint32_t v, int sum) { return (int)__builtin_amdgcn_sad_u8(v, 0u, (uint32_t)sum); }
template <int THREADS>
__device__ __forceinline__ int rows_of_block(const PlanShared &sh, int wv, int &before) {
  const u32x4 c = *(const u32x4 *)sh.wave_cnt[lane_id()];
  int all = 0;
  before = 0;
#pragma unroll
  for (int i = 0; i < THREADS / kWave / 4; ++i) {
    const int n = wv - 4 * i;   // waves of this word that come before
    all = byte_sum(c[i], all);
    before = byte_sum(n >= 4 ? c[i] : n <= 0 ? 0u : c[i] & ~(~0u << (8 * n)), before);
  }
  return all;
}

// The LDS behind PlanShared, if the tables are staged: [hist: E int32 if the load arrays are asked for][table: E + 1 uint16].
extern __shared__ int32_t plan_dyn_lds[];

__global__ __launch_bounds__(kPlanThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void plan_count_kernel(PlanParams p, int staged) {
  __shared__ PlanShared sh;
  const Tokens k = tokens_of_block(p);
  plan_slots<true, kPlanThreads>(p, sh, k, nullptr, staged ? (uint16_t *)plan_dyn_lds : nullptr, blockIdx.x == 0);
  if ((int)threadIdx.x < p.Dn) {
    int before;
    p.counts[(int64_t)blockIdx.x * p.Dn + threadIdx.x] = rows_of_block<kPlanThreads>(sh, 0, before);
  }
  if (p.load_expert) {   // the write kernel accumulates into these with atomics
    const int64_t stride = (int64_t)gridDim.x * kPlanThreads;
    for (int64_t i = (int64_t)blockIdx.x * kPlanThreads + threadIdx.x; i < p.E; i += stride) p.load_expert[i] = 0;
    if (blockIdx.x == 0 && (int)threadIdx.x < p.G) p.load_rank[threadIdx.x] = 0;
    if (blockIdx.x == 0 && (int)threadIdx.x < p.N) p.load_node[threadIdx.x] = 0;
  }
}

// Column d of the count matrix -> exclusive prefix over the workgroups, in place; total -> row nblocks.
__global__ __launch_bounds__(kPlanThreads) void plan_scan_kernel(PlanParams p) {
  __shared__ int32_t wave_tot[kPlanWaves];
  __shared__ int32_t carry;
  const int lane = lane_id(), wv = (int)(threadIdx.x >> 6);
  const int d = blockIdx.x;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int b0 = 0; b0 < p.nblocks; b0 += kPlanThreads) {
    const int b = b0 + (int)threadIdx.x;
    const int v = b < p.nblocks ? p.counts[(int64_t)b * p.Dn + d] : 0;
    int incl = v;
    for (int off = 1; off < kWave; off <<= 1) {
      const int u = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += u;
    }
    if (lane == kWave - 1) wave_tot[wv] = incl;
    __syncthreads();
    int base = carry;
    for (int w = 0; w < wv; ++w) base += wave_tot[w];
    if (b < p.nblocks) p.counts[(int64_t)b * p.Dn + d] = base + incl - v;
    __syncthreads();
    if (threadIdx.x == 0) {
      int tot = 0;
      for (int w = 0; w < kPlanWaves; ++w) tot += wave_tot[w];
      carry += tot;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) p.counts[(int64_t)p.nblocks * p.Dn + d] = carry;
}

// ---- one-launch plan ---------------------------------------------------------------------------
constexpr int kTagShift = 11;   // a workgroup keeps at most 1024 slots per destination: the count takes 11 bits

// The grid-wide step without a separate barrier: a workgroup publishes its per-destination
// counts as 64-bit words (launch tag << 11 | count), one atomic store each, and every workgroup
// reads the whole matrix, waiting on each word until it carries the tag of this launch -- the
// count and its "ready" flag arrive in one word, so no fence orders them.  The tag is 53 bits
// of a value unique to the launch, so what an uninitialised workspace holds cannot pass for it.
// passed[b] is set once workgroup b has read the matrix; workgroup 0 finally waits for all of
// passed and zeroes matrix and flags, so a replay of a captured launch (same tag) starts clean.
// Every wait is bounded by kPlanSpinLimit polls; a wave that gives up makes the workgroup skip
// its writes, flags HM_ERR_HIP and exits.
//
// The chain of dependent memory trips is kept short: the expert -> rank table is staged in LDS while the ids are
// in flight (no dependent lookup), the halo slots are fetched in the same round as the workgroup's own, and what needs no
// other workgroup's counts -- slot_keep, the masks -- is stored while the counts are on their way.
//
// `clean` is set for launches that are captured: a replay carries the same tag, so workgroup 0 waits until all have
// read the matrix (passed) and zeroes both.  A tag that is used once needs no such end, which is a trip to memory
// and back longer than the kernel otherwise is.
enum class PlanMode { kAlone, kFused, kWrite };   // the only workgroup; one launch of several; counts already there

template <PlanMode MODE, int THREADS = kPlanThreads>
__device__ __forceinline__ void plan_body(const PlanParams &p, uint64_t *matrix, uint64_t *passed, uint64_t tag, int staged,
                                          int clean) {
  constexpr bool ALONE = MODE == PlanMode::kAlone, FUSED = MODE == PlanMode::kFused;
  __shared__ PlanShared sh;
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), tid = (int)threadIdx.x;
  const int bid = (int)blockIdx.x;
  const bool loads = p.load_expert != nullptr;
  int32_t *const hist = staged && loads ? plan_dyn_lds : nullptr;
  uint16_t *const table = staged ? (uint16_t *)(plan_dyn_lds + (loads ? p.E : 0)) : nullptr;
  const Tokens k = tokens_of_block(p);
  if (FUSED && bid == 0 && loads) {   // what the atomics of the other workgroups add to: out before this workgroup's counts are
    for (int i = tid; i < p.E; i += kPlanThreads) st_device(p.load_expert + i, 0);
    if (tid < p.G) st_device(p.load_rank + tid, 0);
    if (tid < p.N) st_device(p.load_node + tid, 0);
  }
  const Slot me = plan_slots<false, THREADS>(p, sh, k, hist, table, !(MODE == PlanMode::kWrite) && bid == 0);
  int before;
  const int rows = rows_of_block<THREADS>(sh, wv, before);   // lane: destination
  if (FUSED && wv == 0 && lane < p.Dn) st_device(matrix + (int64_t)bid * p.Dn + lane, (tag << kTagShift) | (uint64_t)rows);

  // ---- while the counts travel: what needs no other workgroup
  if (me.live) {
    if (!me.has_dest) p.slot_row[me.s] = -1;
    p.slot_keep[me.s] = me.keep ? 1 : 0;
  }
  // The masks of the tokens whose first slot is this workgroup's: a lane per token, or eight for tokens of more than sixteen
  // slots, of which there are at most 62.  (One: 16 x 33 slots 8.2 us, eight 7.2; 900 x 64 14.1, 11.1; but 30,000 x 10 20.8, 22.0.)
  const bool by_node = p.level == HM_DEDUP_NODE && !p.dest_map;
  const uint64_t *const ranks = by_node ? sh.other_bytes : sh.dest_bytes, *const nodes = by_node ? sh.dest_bytes : sh.other_bytes;
  if (__builtin_expect(k.words > 2, 0)) {
    const int tok = tid >> 3, wd = tid & 7, t = k.first_token + tok;
    if (tok < k.tokens && t * p.K >= k.first_slot) {
      if (p.rank_mask) {
        const uint64_t mask = mask_of_words<uint64_t>(ranks, k, tok, wd);
        if (wd == 0) p.rank_mask[t] = mask;
      }
      if (p.node_mask) {
        const uint32_t mask = p.dest_map ? 0u : mask_of_words<uint32_t>(nodes, k, tok, wd);
        if (wd == 0) p.node_mask[t] = mask;
      }
    }
  } else if (tid < k.tokens) {
    const int t = k.first_token + tid;
    if (t * p.K >= k.first_slot) {
      if (p.rank_mask) p.rank_mask[t] = mask_of_token<uint64_t>(ranks, k, p.K, tid);
      if (p.node_mask) p.node_mask[t] = p.dest_map ? 0u : mask_of_token<uint32_t>(nodes, k, p.K, tid);
    }
  }
  // The duplicate-free loads of hm_expert_load: the first slot of a token with a rank or a node counts it there.  Where
  // rows are per rank (node) their counts are those of the ranks (nodes) already.
  if (loads && me.has_dest) {
    if (first_in_token(sh.other_bytes, k, me.tok, me.place, me.other))
      atomicAdd(p.level == HM_DEDUP_NODE ? &sh.rank_cnt[me.other] : &sh.node_cnt[me.other], 1);
    if (p.level == HM_DEDUP_NONE && me.first) atomicAdd(&sh.rank_cnt[me.dest], 1);
  }

  // ---- rows of all workgroups and of those before this one, per destination
  int tot = rows, pre = 0;
  if (!ALONE) {
    tot = 0;
    bool ready = true;
    if (FUSED) {   // wave wv reads rows wv, wv + 16, ..., again as a whole wave until every word carries this launch's tag
      for (int spin = 0; spin < kPlanSpinLimit; ++spin) {
        tot = pre = 0;
        bool mine = true;
        if (lane < p.Dn) {
          for (int b0 = wv; b0 < p.nblocks; b0 += 4 * kPlanWaves) {   // four rows in flight
            uint64_t v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int b = b0 + j * kPlanWaves;
              v[j] = b < p.nblocks ? ld_device(matrix + (int64_t)b * p.Dn + lane) : (tag << kTagShift);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              mine = mine && (v[j] >> kTagShift) == tag;
              const int c = (int)(v[j] & ((1u << kTagShift) - 1u));
              tot += c;
              if (b0 + j * kPlanWaves < bid) pre += c;
            }
          }
        }
        ready = __ballot(!mine) == 0ull;
        if (ready) break;
        __builtin_amdgcn_s_sleep(2);
      }
    } else if (lane < p.Dn) {   // an earlier launch left the counts (or, scanned, their prefixes and a row of totals)
      if (p.scanned) {
        if (wv == 0) {
          tot = p.counts[(int64_t)p.nblocks * p.Dn + lane];
          pre = p.counts[(int64_t)bid * p.Dn + lane];
        }
      } else {
        for (int b0 = wv; b0 < p.nblocks; b0 += 8 * kPlanWaves) {   // eight rows in flight
          int c[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int b = b0 + j * kPlanWaves;
            c[j] = b < p.nblocks ? p.counts[(int64_t)b * p.Dn + lane] : 0;
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            tot += c[j];
            if (b0 + j * kPlanWaves < bid) pre += c[j];
          }
        }
      }
    }
    if (tot) atomicAdd(&sh.all_tot[lane], tot);
    if (pre) atomicAdd(&sh.all_pre[lane], pre);
    if (!ready && lane == 0) sh.gave_up = 1;
    __syncthreads();
    tot = sh.all_tot[lane];
    pre = sh.all_pre[lane];
  }
  const bool go = ALONE || sh.gave_up == 0;   // uniform over the workgroup
  if (go) {
    if (FUSED && clean && tid == 0) st_device(passed + bid, tag);
    if (loads) {   // global atomics first: they complete in the shadow of the map stores
      for (int e = tid; hist && e < p.E; e += THREADS) {
        if (ALONE) p.load_expert[e] = hist[e];
        else if (hist[e]) atomicAdd(&p.load_expert[e], hist[e]);
      }
      if (!hist && me.has_dest) atomicAdd(&p.load_expert[me.id], 1);
      if (!ALONE && tid < kWave) {
        const int r = p.level == HM_DEDUP_GPU ? rows : sh.rank_cnt[tid], n = p.level == HM_DEDUP_NODE ? rows : sh.node_cnt[tid];
        if (r) atomicAdd(&p.load_rank[tid], r);
        if (n) atomicAdd(&p.load_node[tid], n);
      }
    }
    if (me.entry == kBadEntry && me.live) flag(p.status, HM_ERR_BAD_ID);

    // ---- rows: the slot that owns a row numbers it and serves the later slots that share it
    const int incl = lane_scan(tot), offset = incl - tot;   // over the destinations (lanes from Dn on hold 0)
    if (bid == 0 && wv == 0 && lane < p.Dn) {
      p.dest_count[lane] = tot;
      p.dest_offset[lane] = offset;
      if (lane == p.Dn - 1) p.dest_offset[p.Dn] = incl;
    }
    const int row = __shfl(offset + pre + before, me.dest & (kWave - 1), kWave) + me.pos;
    if (me.keep) {
      p.slot_row[me.s] = row;
      float wsum = me.w;
      if (p.level != HM_DEDUP_NONE) {
        const uint64_t *const token = sh.dest_bytes + me.tok * k.words;
        const uint64_t same = repeated(me.dest);
        uint64_t later = ~0xFFull << (8 * (me.place & 7));   // the bytes behind mine
#pragma unroll 1
        for (int wd = me.place >> 3; wd < k.words; ++wd, later = ~0ull) {
#pragma unroll 1
          for (uint64_t m = equal_bytes(token[wd], same) & later; m; m &= m - 1) {
            const int ahead = wd * 8 + (__builtin_ctzll(m) >> 3) - me.place;
            p.slot_row[me.s + ahead] = row;
            wsum = wsum + sh.weight[tid + ahead];  // ascending k, fp32
          }
        }
      }
      if (row < p.row_capacity) {
        p.row_token[row] = k.first_token + me.tok;
        p.row_weight[row] = wsum;
      } else {
        flag(p.status, HM_ERR_CAPACITY);
      }
    }
  } else if (tid == 0) {
    flag(p.status, HM_ERR_HIP);
  }
  if (ALONE && loads) {   // the other modes have had a barrier since the tokens were counted
    __syncthreads();
    if (tid < p.G) p.load_rank[tid] = p.level == HM_DEDUP_GPU ? rows : sh.rank_cnt[tid];
    if (tid < p.N) p.load_node[tid] = p.level == HM_DEDUP_NODE ? rows : sh.node_cnt[tid];
  }

  // ---- workgroup 0 leaves matrix and flags clean (also when a wait gave up: the status word says so)
  if (FUSED && clean && bid == 0) {
    if (wv == 0 && go) {
      bool ok = true;
      for (int spin = 0; spin < kPlanSpinLimit; ++spin) {
        ok = true;
        for (int b = lane; b < p.nblocks; b += kWave) ok = ok && ld_device(passed + b) == tag;
        if (__ballot(!ok) == 0ull) break;
        __builtin_amdgcn_s_sleep(2);
      }
      if (__ballot(!ok) != 0ull && lane == 0) flag(p.status, HM_ERR_HIP);
    }
    __syncthreads();
    for (int i = tid; i < p.nblocks * p.Dn; i += kPlanThreads) st_device(matrix + i, 0ull);
    for (int b = tid; b < p.nblocks; b += kPlanThreads) st_device(passed + b, 0ull);
  }
}

// The one-launch plan.  It runs one workgroup per CU at the sizes it is used for, so it takes the
// scalar registers the compiler wants (106: the many pointers of PlanParams).
__global__ __launch_bounds__(kPlanThreads) void plan_fused_kernel(PlanParams p, uint64_t *matrix, uint64_t *passed,
                                                                  uint64_t tag, int staged, int clean) {
  plan_body<PlanMode::kFused>(p, matrix, passed, tag, staged, clean);
}

// A plan of one workgroup: nothing to wait for, nothing to clear, no atomics outside LDS.  Few slots take few waves,
// which issue their instructions one after the other (graphs of twenty calls, 1,024 lanes -> as many as the slots want, us: 16 x 8
// slots 4.45 -> 4.16, 64 x 8 4.60 -> 4.31, 300 x 3 without dedup 4.78 -> 4.40, at rank level 5.06 -> 4.69).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void plan_alone_kernel(PlanParams p) {
  plan_body<PlanMode::kAlone, THREADS>(p, nullptr, nullptr, 0, 1, 0);
}

// The last launch of a large plan: the same body without the grid-wide wait.  Held to 96 scalar
// registers, i.e. eight waves per SIMD, so that two workgroups fit a CU and the 512 workgroups of a
// 64 Ki-token layer run in one round (thirty-odd scalars then live in vector lanes, which is
// cheaper than a second round).
__global__ __launch_bounds__(kPlanThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void plan_write_kernel(PlanParams p,
                                                                                                      int staged) {
  plan_body<PlanMode::kWrite>(p, nullptr, nullptr, 0, staged, 0);
}

// Table of one hop for a (parent, child) pair of group cuts: purely elementwise.
__global__ __launch_bounds__(kPlanThreads) void level_dest_map_kernel(const int32_t *__restrict__ expert_to_rank, int E,
                                                                       int G, int my_rank, int ranks_per_parent,
                                                                       int ranks_per_child, int children_per_parent,
                                                                       int32_t *__restrict__ dest_map,
                                                                       int32_t *__restrict__ num_dest) {
  const int e = blockIdx.x * kPlanThreads + threadIdx.x;
  if (e == 0) *num_dest = children_per_parent;
  if (e >= E) return;
  const int g = expert_to_rank[e];
  int v;
  if ((unsigned)g >= (unsigned)G) v = -2;
  else if (g / ranks_per_parent != my_rank / ranks_per_parent) v = -1;
  else v = (g / ranks_per_child) % children_per_parent;
  dest_map[e] = v;
}

// Destination table of a receiver stage: one workgroup walks the E experts in chunks of 1024 and
// numbers the experts placed on `my_rank` with a ballot scan, so local indices ascend with the
// expert id.
__global__ __launch_bounds__(kPlanThreads) void recv_dest_map_kernel(const int32_t *__restrict__ expert_to_rank, int E,
                                                                      int G, int R, int my_rank, int stage,
                                                                      int32_t *__restrict__ dest_map,
                                                                      int32_t *__restrict__ num_dest) {
  __shared__ int32_t wave_cnt[kPlanWaves];
  __shared__ int32_t base;
  const int lane = lane_id(), wv = (int)(threadIdx.x >> 6);
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int e0 = 0; e0 < E; e0 += kPlanThreads) {
    const int e = e0 + (int)threadIdx.x;
    int g = -1;
    if (e < E) {
      g = expert_to_rank[e];
      if ((unsigned)g >= (unsigned)G) g = -2;
    }
    const bool mine = g == my_rank;
    const uint64_t b = __ballot(mine);
    if (lane == 0) wave_cnt[wv] = __popcll(b);
    __syncthreads();
    int before = base;
    for (int w = 0; w < wv; ++w) before += wave_cnt[w];
    if (e < E) {
      int v;
      if (g == -2) v = -2;
      else if (stage == HM_RECV_INTRA_NODE) v = (g / R == my_rank / R) ? g % R : -1;
      else v = mine ? before + __popcll(b & ((1ull << lane) - 1ull)) : -1;
      dest_map[e] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int tot = 0;
      for (int w = 0; w < kPlanWaves; ++w) tot += wave_cnt[w];
      base += tot;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *num_dest = stage == HM_RECV_INTRA_NODE ? R : base;
}

static inline int32_t plan_blocks(int64_t nslots) {
  const int64_t b = (nslots + kPlanThreads - 1) / kPlanThreads;
  return (int32_t)(b < 1 ? 1 : b);
}

// Workspace: the count matrix [workgroups + 1][Dn] int32 of the multi-launch kernels, then
// (8-byte aligned) what the one-launch kernel uses instead: a matrix of [workgroups][Dn] tagged
// 64-bit words and one 64-bit flag per workgroup.
static inline size_t plan_counts_bytes(int64_t nslots, int Dn) {
  const size_t b = ((size_t)plan_blocks(nslots) + 1) * (size_t)Dn * sizeof(int32_t);
  return (b + 7) & ~(size_t)7;
}
static inline size_t plan_workspace(int64_t nslots, int Dn) {
  const int32_t nb = plan_blocks(nslots);
  const size_t fused = nb <= kPlanFusedMaxBlocks ? ((size_t)nb * (size_t)Dn + (size_t)nb) * sizeof(uint64_t) : 0;
  return plan_counts_bytes(nslots, Dn) + fused;
}

// Workgroups of plan_fused_kernel that can be resident together on the current device (0 if that
// cannot be established: the multi-launch path is always available).
static inline int fused_capacity() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int v = cached[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    int cus = 0, per_cu = 0;
    v = -1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, plan_fused_kernel, kPlanThreads,
                                                     kPlanStagedExperts * 6 + 16) == hipSuccess &&
        cus > 0 && per_cu > 0)
      v = cus * per_cu;
    cached[dev].store(v, std::memory_order_relaxed);
  }
  return v > 0 ? v : 0;
}

// 53 bits no earlier launch of this process has used and stale memory is unlikely to hold; never 0.
static inline uint64_t next_tag() {
  static std::atomic<uint64_t> counter{0};
  static std::once_flag seeded;
  std::call_once(seeded, [] {
    uint64_t z = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ ((uint64_t)getpid() << 40);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    counter.store(z ^ (z >> 31), std::memory_order_relaxed);
  });
  const uint64_t mask = (1ull << 53) - 1ull;
  uint64_t e = (counter.fetch_add(1, std::memory_order_relaxed) + 1) & mask;
  if (e == 0) e = (counter.fetch_add(1, std::memory_order_relaxed) + 1) & mask;
  return e;
}

// Whether launches on the stream go into a graph; also when that cannot be told.
static inline int is_captured(hipStream_t stream) {
  hipStreamCaptureStatus now = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &now) == hipSuccess) return now != hipStreamCaptureStatusNone ? 1 : 0;
  if (hipPeekAtLastError() != hm_pending_at_entry) (void)hipGetLastError();   // not a failed launch
  return 1;
}

// Largest plan, in workgroups, that takes the one-launch kernel (hm_plan_one_launch_limit).
static std::atomic<int> one_launch_limit{kPlanFusedMaxBlocks};

// One launch when the plan is small enough, else count -> (scan) -> write, on `stream`;
// p.nblocks, p.Dn and p.counts are set.
static inline hm_status launch_plan(PlanParams &p, hipStream_t stream) {
  const bool loads = p.load_expert != nullptr;
  p.N = p.G / p.R;
  p.k_recip = p.K > 1 ? ~0ull / (uint64_t)p.K + 1 : 0;
  p.k_recip22 = ((1u << 22) + (uint32_t)p.K - 1u) / (uint32_t)p.K;
  p.r_recip16 = (65536u + (uint32_t)p.R - 1u) / (uint32_t)p.R;
  const int staged = p.E <= kPlanStagedExperts ? 1 : 0;   // tables (and histogram) in LDS
  const unsigned table_lds = staged ? (2u * ((unsigned)p.E + 1u) + 15u) & ~15u : 0u;
  const unsigned lds = staged && loads ? (unsigned)p.E * sizeof(int32_t) + table_lds : table_lds;
  if (p.nblocks == 1 && staged) {
    if (p.nslots <= 256) hipLaunchKernelGGL(plan_alone_kernel<256>, dim3(1), dim3(256), lds, stream, p);
    else if (p.nslots <= 512) hipLaunchKernelGGL(plan_alone_kernel<512>, dim3(1), dim3(512), lds, stream, p);
    else hipLaunchKernelGGL(plan_alone_kernel<kPlanThreads>, dim3(1), dim3(kPlanThreads), lds, stream, p);
    return hm_launch_status();
  }
  if (p.nblocks <= one_launch_limit.load(std::memory_order_relaxed) && p.nblocks <= fused_capacity()) {
    p.scanned = 0;
    uint64_t *matrix = (uint64_t *)((char *)p.counts + plan_counts_bytes(p.nslots, p.Dn));
    hipLaunchKernelGGL(plan_fused_kernel, dim3(p.nblocks), dim3(kPlanThreads), lds, stream, p, matrix,
                       matrix + (size_t)p.nblocks * p.Dn, next_tag(), staged, is_captured(stream));
    return hm_launch_status();
  }
  p.scanned = (int64_t)p.nblocks * p.Dn >= kPlanScanMinEntries ? 1 : 0;
  hipLaunchKernelGGL(plan_count_kernel, dim3(p.nblocks), dim3(kPlanThreads), table_lds, stream, p, staged);
  if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  if (p.scanned) {
    hipLaunchKernelGGL(plan_scan_kernel, dim3(p.Dn), dim3(kPlanThreads), 0, stream, p);
    if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  }
  // the same kernel without its grid-wide wait: the counts are complete
  hipLaunchKernelGGL(plan_write_kernel, dim3(p.nblocks), dim3(kPlanThreads), lds, stream, p, staged);
  return hm_launch_status();
}

}  // namespace hm

extern "C" int32_t hm_plan_one_launch_capacity(void) { return hm::fused_capacity(); }

extern "C" int32_t hm_plan_one_launch_limit(int32_t workgroups) {
  const int v = workgroups < 0 ? 0 : workgroups > hm::kPlanFusedMaxBlocks ? hm::kPlanFusedMaxBlocks : workgroups;
  return hm::one_launch_limit.exchange(v, std::memory_order_relaxed);
}

extern "C" size_t hm_plan_workspace_bytes(int32_t T, int32_t K, int32_t E, hm_topology topo, hm_dedup_level level) {
  if (E < 1 || hm_check_tk(T, K) != HM_OK || hm_check_topology(topo) != HM_OK) return 0;
  if (level != HM_DEDUP_NONE && level != HM_DEDUP_GPU && level != HM_DEDUP_NODE) return 0;
  const int Dn = level == HM_DEDUP_NODE ? topo.nodes : topo.nodes * topo.ranks_per_node;
  return hm::plan_workspace((int64_t)T * K, Dn);
}

// Argument checks and launches of hm_plan; `counts` is the count matrix (caller's workspace or the
// library's static scratch), already known to be large enough.
static hm_status plan_on_counts(const int32_t *topk_ids, const float *topk_weights, const int32_t *expert_to_rank,
                                int32_t T, int32_t K, int32_t E, hm_topology topo, hm_dedup_level level, hm_plan_out *out,
                                int32_t *counts, void *hip_stream) {
  hm::PlanParams p;
  p.ids = topk_ids;
  p.weights = topk_weights;
  p.expert_to_rank = expert_to_rank;
  p.dest_map = nullptr;
  p.T = T;
  p.K = K;
  p.E = E;
  p.R = topo.ranks_per_node;
  p.G = topo.nodes * topo.ranks_per_node;
  p.Dn = level == HM_DEDUP_NODE ? topo.nodes : p.G;
  p.level = (int32_t)level;
  p.nslots = (int32_t)((int64_t)T * K);
  p.nblocks = hm::plan_blocks(p.nslots);
  p.row_capacity = out->row_capacity;
  p.counts = counts;
  p.dest_count = out->dest_count;
  p.dest_offset = out->dest_offset;
  p.row_token = out->row_token;
  p.slot_row = out->slot_row;
  p.slot_keep = out->slot_keep;
  p.row_weight = out->row_weight;
  p.rank_mask = out->rank_mask;
  p.node_mask = out->node_mask;
  p.status = out->status;
  p.load_expert = out->load_expert;
  p.load_rank = out->load_rank;
  p.load_node = out->load_node;
  out->num_dest = p.Dn;
  out->max_rows_per_token = level == HM_DEDUP_NONE ? K : (K < p.Dn ? K : p.Dn);
  return hm::launch_plan(p, (hipStream_t)hip_stream);
}

static hm_status check_plan_args(const int32_t *topk_ids, const float *topk_weights, const int32_t *expert_to_rank,
                                 int32_t T, int32_t K, int32_t E, hm_topology topo, hm_dedup_level level,
                                 const hm_plan_out *out) {
  if (!out || !expert_to_rank) return HM_ERR_NULL;
  if (!out->dest_count || !out->dest_offset || !out->row_token || !out->slot_row || !out->slot_keep ||
      !out->row_weight || !out->status)
    return HM_ERR_NULL;
  hm_status st = hm_check_tk(T, K);
  if (st != HM_OK) return st;
  if (E < 1 || out->row_capacity < 0) return HM_ERR_SHAPE;
  if (T > 0 && (!topk_ids || !topk_weights)) return HM_ERR_NULL;
  if (out->load_expert && (!out->load_rank || !out->load_node)) return HM_ERR_NULL;
  if (!out->load_expert && (out->load_rank || out->load_node)) return HM_ERR_NULL;
  st = hm_check_topology(topo);
  if (st != HM_OK) return st;
  if (level != HM_DEDUP_NONE && level != HM_DEDUP_GPU && level != HM_DEDUP_NODE) return HM_ERR_LEVEL;
  return HM_OK;
}

extern "C" hm_status hm_plan(const int32_t *topk_ids, const float *topk_weights, const int32_t *expert_to_rank,
                             int32_t T, int32_t K, int32_t E, hm_topology topo, hm_dedup_level level,
                             hm_plan_out *out, void *workspace, size_t workspace_bytes, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!workspace) return HM_ERR_NULL;
  hm_status st = check_plan_args(topk_ids, topk_weights, expert_to_rank, T, K, E, topo, level, out);
  if (st != HM_OK) return st;
  if (workspace_bytes < hm_plan_workspace_bytes(T, K, E, topo, level)) return HM_ERR_WORKSPACE;
  return plan_on_counts(topk_ids, topk_weights, expert_to_rank, T, K, E, topo, level, out, (int32_t *)workspace,
                        hip_stream);
}

// ---- hm_plan_static: hm_plan for callers that cannot hand over (or allocate) a workspace ----------
// The count matrix lives in a file-scope device array.  In host code the array's name is only a
// stand-in for the symbol: its device address is looked up once per device and that pointer is
// what the kernels receive.
namespace hm {
constexpr size_t kPlanStaticBytes = (size_t)1 << 20;   // 1 MiB per GPU, held until the process ends
constexpr int kPlanStaticDevices = 64;
static __device__ __align__(256) unsigned char plan_static_scratch[kPlanStaticBytes];
static std::mutex plan_static_lock;
static void *plan_static_ptr[kPlanStaticDevices];   // device address of the array on each GPU, 0 = not asked yet

// Device address of the current GPU's copy of the scratch array (nullptr on a HIP error).
static void *plan_static_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kPlanStaticDevices) return nullptr;
  std::lock_guard<std::mutex> hold(plan_static_lock);
  if (!plan_static_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(plan_static_scratch)) != hipSuccess) return nullptr;
    plan_static_ptr[dev] = ptr;
  }
  return plan_static_ptr[dev];
}
}  // namespace hm

extern "C" size_t hm_plan_static_max_bytes(void) { return hm::kPlanStaticBytes; }

extern "C" hm_status hm_plan_static(const int32_t *topk_ids, const float *topk_weights, const int32_t *expert_to_rank,
                                    int32_t T, int32_t K, int32_t E, hm_topology topo, hm_dedup_level level,
                                    hm_plan_out *out, void *hip_stream) {
  HM_ENTRY_SCOPE;
  hm_status st = check_plan_args(topk_ids, topk_weights, expert_to_rank, T, K, E, topo, level, out);
  if (st != HM_OK) return st;
  if (hm_plan_workspace_bytes(T, K, E, topo, level) > hm::kPlanStaticBytes) return HM_ERR_WORKSPACE;
  void *counts = hm::plan_static_address();
  if (!counts) return HM_ERR_HIP;
  // Nothing in the matrix has to start at zero: the count kernel overwrites every entry the later
  // kernels read, so the previous call's contents are harmless.
  return plan_on_counts(topk_ids, topk_weights, expert_to_rank, T, K, E, topo, level, out, (int32_t *)counts,
                        hip_stream);
}

extern "C" size_t hm_plan_mapped_workspace_bytes(int32_t rows, int32_t K, int32_t num_dest) {
  if (hm_check_tk(rows, K) != HM_OK || num_dest < 1 || num_dest > 64) return 0;
  return hm::plan_workspace((int64_t)rows * K, num_dest);
}

extern "C" hm_status hm_plan_mapped(const int32_t *row_ids, const float *row_weights, const int32_t *dest_map,
                                    int32_t rows, int32_t K, int32_t E, int32_t num_dest, int32_t dedup, hm_plan_out *out,
                                    void *workspace, size_t workspace_bytes, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!out || !dest_map || !workspace) return HM_ERR_NULL;
  if (!out->dest_count || !out->dest_offset || !out->row_token || !out->slot_row || !out->slot_keep ||
      !out->row_weight || !out->status)
    return HM_ERR_NULL;
  hm_status st = hm_check_tk(rows, K);
  if (st != HM_OK) return st;
  if (E < 1 || out->row_capacity < 0) return HM_ERR_SHAPE;
  if (num_dest < 1 || num_dest > 64) return HM_ERR_TOPOLOGY;
  if (rows > 0 && (!row_ids || !row_weights)) return HM_ERR_NULL;
  if (workspace_bytes < hm_plan_mapped_workspace_bytes(rows, K, num_dest)) return HM_ERR_WORKSPACE;

  hm::PlanParams p;
  p.ids = row_ids;
  p.weights = row_weights;
  p.expert_to_rank = nullptr;
  p.dest_map = dest_map;
  p.T = rows;
  p.K = K;
  p.E = E;
  p.R = 1;
  p.G = num_dest;
  p.Dn = num_dest;
  p.level = dedup ? (int32_t)HM_DEDUP_GPU : (int32_t)HM_DEDUP_NONE;
  p.nslots = (int32_t)((int64_t)rows * K);
  p.nblocks = hm::plan_blocks(p.nslots);
  p.row_capacity = out->row_capacity;
  p.counts = (int32_t *)workspace;
  p.dest_count = out->dest_count;
  p.dest_offset = out->dest_offset;
  p.row_token = out->row_token;
  p.slot_row = out->slot_row;
  p.slot_keep = out->slot_keep;
  p.row_weight = out->row_weight;
  p.rank_mask = out->rank_mask;
  p.node_mask = out->node_mask;
  p.status = out->status;
  p.load_expert = p.load_rank = p.load_node = nullptr;   // the fused loads need the rank placement
  out->num_dest = num_dest;
  out->max_rows_per_token = 0;   // a hop table may leave most slots without a copy: no useful bound

  return hm::launch_plan(p, (hipStream_t)hip_stream);
}

extern "C" hm_status hm_recv_dest_map(const int32_t *expert_to_rank, int32_t E, hm_topology topo, int32_t my_rank,
                                      hm_recv_stage stage, int32_t *dest_map, int32_t *num_dest, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!expert_to_rank || !dest_map || !num_dest) return HM_ERR_NULL;
  if (E < 1) return HM_ERR_SHAPE;
  hm_status st = hm_check_topology(topo);
  if (st != HM_OK) return st;
  const int G = topo.nodes * topo.ranks_per_node;
  if (my_rank < 0 || my_rank >= G) return HM_ERR_TOPOLOGY;
  if (stage != HM_RECV_INTRA_NODE && stage != HM_RECV_LOCAL_EXPERTS) return HM_ERR_LEVEL;
  hipLaunchKernelGGL(hm::recv_dest_map_kernel, dim3(1), dim3(hm::kPlanThreads), 0, (hipStream_t)hip_stream,
                     expert_to_rank, E, G, topo.ranks_per_node, my_rank, (int)stage, dest_map, num_dest);
  return hm_launch_status();
}

extern "C" hm_status hm_level_dest_map(const int32_t *expert_to_rank, int32_t E, int32_t G, int32_t my_rank,
                                       int32_t parent_groups, int32_t child_groups, int32_t *dest_map, int32_t *num_dest,
                                       void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!expert_to_rank || !dest_map || !num_dest) return HM_ERR_NULL;
  if (E < 1) return HM_ERR_SHAPE;
  if (G < 1 || G > 64 || my_rank < 0 || my_rank >= G) return HM_ERR_TOPOLOGY;
  if (parent_groups < 1 || child_groups < parent_groups || child_groups > G) return HM_ERR_TOPOLOGY;
  if (child_groups % parent_groups != 0 || G % child_groups != 0) return HM_ERR_TOPOLOGY;
  const int blocks = (E + hm::kPlanThreads - 1) / hm::kPlanThreads;
  hipLaunchKernelGGL(hm::level_dest_map_kernel, dim3(blocks), dim3(hm::kPlanThreads), 0, (hipStream_t)hip_stream,
                     expert_to_rank, E, G, my_rank, G / parent_groups, G / child_groups, child_groups / parent_groups,
                     dest_map, num_dest);
  return hm_launch_status();
}

extern "C" hm_status hm_plan_status(hm_plan_out *plan, int64_t *total_rows, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!plan || !plan->status || !plan->dest_offset) return HM_ERR_NULL;
  if (plan->num_dest < 1 || plan->num_dest > 64) return HM_ERR_SHAPE;
  hipStream_t stream = (hipStream_t)hip_stream;
  int32_t host[2] = {0, 0};
  if (hipMemcpyAsync(&host[0], plan->status, sizeof(int32_t), hipMemcpyDeviceToHost, stream) != hipSuccess)
    return HM_ERR_HIP;
  if (hipMemcpyAsync(&host[1], plan->dest_offset + plan->num_dest, sizeof(int32_t), hipMemcpyDeviceToHost,
                     stream) != hipSuccess)
    return HM_ERR_HIP;
  if (hipStreamSynchronize(stream) != hipSuccess) return HM_ERR_HIP;
  if (total_rows) *total_rows = host[1];
  plan->expected_rows = host[1];   // what the row kernels size their launches by
  return (hm_status)host[0];
}

extern "C" const char *hm_status_string(hm_status s) {
  switch (s) {
    case HM_OK: return "ok";
    case HM_ERR_NULL: return "null pointer";
    case HM_ERR_SHAPE: return "bad shape";
    case HM_ERR_TOPOLOGY: return "bad topology (need 1..32 nodes, at most 64 ranks)";
    case HM_ERR_LEVEL: return "bad dedup level";
    case HM_ERR_WORKSPACE: return "workspace too small (hm_plan_static: sizes beyond its static scratch)";
    case HM_ERR_CAPACITY: return "row index beyond the caller's row buffers";
    case HM_ERR_BAD_ID: return "expert id or rank out of range";
    case HM_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}
