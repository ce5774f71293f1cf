// Hierarchical expert swap (HierMoE Section IV): the swap tensor Z and the selection of Eq.(8)-(11).
//
// Z[r][c][:] is the vector of duplicate-free per-group token counts after experts r and c trade
// places.  A swap can only change the two groups involved, and by how much follows from three
// small co-occurrence tables over the tokens:
//   L0[a]    tokens selecting a                      CG[a][g]  ... that also select something in g
//   L[a]     tokens where a is alone in its group    C[a][b]   ... that also select b
// For g_r != g_c:  Z[r][c][g_c] = base[g_c] + (L0[r] - CG[r][g_c]) - (L[c] - C[c][r])   and the same
// with r and c exchanged for g_r: no O(T K E) walk over all unselected experts, and the per-pair
// work is an embarrassingly parallel E^2 ng kernel.  The tables come from int8 matrix products on
// the matrix cores for E <= 512 (further down), from O(T K (K + ng)) atomic updates, one lane per
// routing slot, beyond that, for E > 256 with more than eight slots per token, and where the products would have
// too little to do (atomics_pay).
#include "hm_device.h"

namespace hm {

constexpr int kSwapThreads = 256;
constexpr int kSelectThreads = 256;    // Q per pair: fp64 pow-heavy, one wave per term of Eq.(8)
constexpr int kSelectPairs = kWave;
constexpr int kFactorThreads = 1024;   // the co-occurrence pass: 16 waves share one set of LDS tables
constexpr int kSwapLds = 30720;   // most ints of LDS for L0 and every cut's L + CG (120 KiB); larger sets stay in global memory
constexpr int kSwapCopiesMax = 32;   // private copies of C: popular expert pairs would otherwise serialise on one address
constexpr int kMaxCuts = 4;       // group cuts handled by one pass over the tokens

// One pass serves up to kMaxCuts cuts of the ranks into groups: everything that does not depend on
// the cut (ids, placement lookups, which slots repeat an expert) is done once.
struct SwapParams {
  const int32_t *ids;
  const int32_t *expert_to_rank;
  int32_t T, K, E, G;
  int32_t sub;      // lanes per token in the co-occurrence pass: the power of two >= K
  int32_t ncuts;
  int32_t use_lds;  // L0 / L / CG of all cuts accumulate in LDS
  int32_t copies;   // private copies of each C
  int32_t ng[kMaxCuts], per[kMaxCuts];
  uint32_t ng_reciprocal[kMaxCuts];   // ceil(2^32 / ng), for the division by ng in swap_build_kernel (unused when ng = 1)
  uint32_t per_reciprocal[kMaxCuts];  // ceil(2^32 / per), 0 when per = 1
  uint32_t quad_reciprocal[kMaxCuts]; // ceil(2^32 / (ng / 4))
  int32_t quads[kMaxCuts];            // swap_build_kernel takes four groups per lane
  int32_t build_blocks[kMaxCuts];     // column blocks of swap_build_kernel per cut
  int32_t lds_off[kMaxCuts];   // ints: where cut c's [L (E) | CG (E * ng)] starts in LDS; L0 is at 0
  int32_t *L0;                 // [E]                                  (workspace, shared by the cuts)
  int32_t *base[kMaxCuts];     // [64]                                 (workspace, per cut)
  int32_t *L[kMaxCuts];        // [E]
  int32_t *CG[kMaxCuts];       // [E][ng]
  int32_t *C[kMaxCuts];        // [copies][E][E]
  int32_t *CT[kMaxCuts];       // [E][E]   C transposed   } matrix path only: swap_build_kernel then reads
  int32_t *CGT[kMaxCuts];      // [ng][E]  CG transposed  } along rows whichever expert of a pair a lane needs
  int32_t cg_by_group[kMaxCuts];   // whether there is room for CGT; else CGT is CG itself, [E][ng]
  int32_t transposed;
  int32_t *Z[kMaxCuts];
  int32_t *ws;                 // start of the workspace and its size in ints (cleared first)
  int64_t ws_ints;
  int32_t *status;
};

__global__ __launch_bounds__(kSwapThreads) void swap_clear_kernel(SwapParams p) {
  const int64_t i = (int64_t)blockIdx.x * kSwapThreads + threadIdx.x;
  if (i < p.ws_ints) p.ws[i] = 0;
  if (i == 0 && p.status) *p.status = 0;
}

// One lane per routing slot: the K slots of a token sit in a sub-group of `sub` = 2^ceil(log2 K)
// consecutive lanes (64 / sub tokens per wave) and learn about each other through shuffles, so the
// per-token work -- K expert updates, K * groups and up to K * K co-occurrence updates -- is spread
// over K lanes instead of being a serial loop of one lane.
__global__ __launch_bounds__(kFactorThreads) void swap_factors_kernel(SwapParams p) {
  extern __shared__ int32_t lds[];   // L0 and every cut's L + CG, sized by the launch
  __shared__ int32_t base_cnt[kMaxCuts][kWave];
  __shared__ uint8_t group_of[kMaxCuts][kWave];   // rank -> group under each cut
  if (p.use_lds) {
    const int used = p.lds_off[p.ncuts - 1] + p.E * (p.ng[p.ncuts - 1] + 1);
    for (int i = threadIdx.x; i < used; i += kFactorThreads) lds[i] = 0;
  }
  if (threadIdx.x < kMaxCuts * kWave) {
    const int c = threadIdx.x / kWave, r = threadIdx.x % kWave;
    base_cnt[c][r] = 0;
    group_of[c][r] = (uint8_t)(c < p.ncuts ? r / p.per[c] : 0);
  }
  __syncthreads();

  const int lane = lane_id();
  const int k = lane & (p.sub - 1);        // my slot in the token
  const int sub0 = lane & ~(p.sub - 1);    // first lane of my token's sub-group
  const int tokens_per_wave = kWave / p.sub;
  const int64_t wave = (int64_t)blockIdx.x * (kFactorThreads / kWave) + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * (kFactorThreads / kWave);
  const int64_t per_round = nwaves * tokens_per_wave;
  const int64_t rounds = ((int64_t)p.T + per_round - 1) / per_round;
  const int64_t copy_off = (int64_t)(blockIdx.x & (p.copies - 1)) * p.E * p.E;
  int my_base[kMaxCuts] = {0, 0, 0, 0};
  for (int64_t it = 0; it < rounds; ++it) {
    const int64_t t = (it * nwaves + wave) * tokens_per_wave + lane / p.sub;
    int a = -1, g = -1;   // my expert and its rank; -1 when the slot is empty, dropped or invalid
    if (t < p.T && k < p.K) {
      const int id = p.ids[t * p.K + k];
      const int r = rank_of(p.expert_to_rank, p.E, p.G, id);
      if (r == -1) flag(p.status, HM_ERR_BAD_ID);
      if (r >= 0) {
        a = id;
        g = r;
      }
    }
    // the selected experts form a set: `first` marks the first valid occurrence of each
    bool first = a >= 0;
    uint64_t gm[kMaxCuts] = {0, 0, 0, 0};   // groups the token touches, per cut
    for (int k1 = 0; k1 < p.K; ++k1) {
      const int a1 = __shfl(a, sub0 + k1, kWave);
      const int g1 = __shfl(g, sub0 + k1, kWave);
      if (k1 < k && a1 == a) first = false;
      if (g1 >= 0) {
#pragma unroll
        for (int c = 0; c < kMaxCuts; ++c)
          if (c < p.ncuts) gm[c] |= 1ull << group_of[c][g1];
      }
    }
    int in_group[kMaxCuts] = {0, 0, 0, 0};   // distinct selected experts in my expert's group
    for (int k1 = 0; k1 < p.K; ++k1) {
      const int f1 = __shfl((int)first, sub0 + k1, kWave);
      const int g1 = __shfl(g, sub0 + k1, kWave);
      if (f1 && g >= 0) {
#pragma unroll
        for (int c = 0; c < kMaxCuts; ++c)
          if (c < p.ncuts) in_group[c] += group_of[c][g1] == group_of[c][g] ? 1 : 0;
      }
    }
    bool alone[kMaxCuts];
#pragma unroll
    for (int c = 0; c < kMaxCuts; ++c) alone[c] = c < p.ncuts && first && in_group[c] == 1;
    if (first) {
      if (p.use_lds) atomicAdd(&lds[a], 1);
      else atomicAdd(&p.L0[a], 1);
#pragma unroll
      for (int c = 0; c < kMaxCuts; ++c) {
        if (c < p.ncuts) {
          int32_t *tL = p.use_lds ? lds + p.lds_off[c] : p.L[c];
          int32_t *tCG = p.use_lds ? lds + p.lds_off[c] + p.E : p.CG[c];
          if (alone[c]) atomicAdd(&tL[a], 1);
          for (uint64_t m = gm[c]; m; m &= m - 1) atomicAdd(&tCG[a * p.ng[c] + __builtin_ctzll(m)], 1);
        }
      }
    }
    // C[a1][b] += 1 for every expert a1 of the token that is alone in its group and every other
    // selected expert b.  The lane of b issues the update, so the lanes of a token hit one row of
    // C per step (a few cache lines) rather than one column (a line per lane).
    int alone_mask = 0;
#pragma unroll
    for (int c = 0; c < kMaxCuts; ++c) alone_mask |= alone[c] ? 1 << c : 0;
    for (int k1 = 0; k1 < p.K; ++k1) {
      const int a1 = __shfl(a, sub0 + k1, kWave);
      const int m1 = __shfl(alone_mask, sub0 + k1, kWave);
      if (first && m1 && a1 != a) {
#pragma unroll
        for (int c = 0; c < kMaxCuts; ++c)
          if (m1 & (1 << c)) atomicAdd(&p.C[c][copy_off + (int64_t)a1 * p.E + a], 1);
      }
    }
    const bool leader = k == 0 && t < p.T;   // one lane per token counts the token's groups
#pragma unroll
    for (int c = 0; c < kMaxCuts; ++c) {
      if (c < p.ncuts) {
        for (int j = 0; j < p.ng[c]; ++j) {
          const uint64_t b = __ballot(leader && ((gm[c] >> j) & 1ull));
          if (lane == j) my_base[c] += __popcll(b);
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kMaxCuts; ++c)
    if (c < p.ncuts && lane < p.ng[c] && my_base[c]) atomicAdd(&base_cnt[c][lane], my_base[c]);
  __syncthreads();
  for (int c = 0; c < p.ncuts; ++c) {
    if ((int)threadIdx.x < p.ng[c] && base_cnt[c][threadIdx.x]) atomicAdd(&p.base[c][threadIdx.x], base_cnt[c][threadIdx.x]);
    if (p.use_lds) {
      const int32_t *sL = lds + p.lds_off[c], *sCG = sL + p.E;
      for (int i = threadIdx.x; i < p.E; i += kFactorThreads)
        if (sL[i]) atomicAdd(&p.L[c][i], sL[i]);
      for (int i = threadIdx.x; i < p.E * p.ng[c]; i += kFactorThreads)
        if (sCG[i]) atomicAdd(&p.CG[c][i], sCG[i]);
    }
  }
  if (p.use_lds)
    for (int i = threadIdx.x; i < p.E; i += kFactorThreads)
      if (lds[i]) atomicAdd(&p.L0[i], lds[i]);
}

// ---------------------------------------------------------------------------------------------
// The same tables as contractions over the tokens (E <= 512).
//
// With S[t][a] = 1 when token t selects expert a, A[t][a] = 1 when a is moreover the only selected
// expert of its group, and M[t][g] = 1 when t selects something in group g (all 0/1 bytes):
//   C  = A^T S   (its diagonal is L)        CG = S^T M   (L0[a] = CG[a][group of a])
// so the read-modify-write updates of popular expert pairs, which serialise on one address, become
// int8 matrix products with int32 accumulators held in registers.  A workgroup takes one cut, a contiguous chunk of
// the tokens and a panel of columns of C, builds the three indicator tiles for 128 tokens at a time in LDS
// (expert-major, so that a lane's MFMA operand is 16 contiguous bytes), and stores its partial tables with plain
// stores; a second kernel sums the chunks.  (With many tokens, or E > 256, for which the workspace has no room
// for partial tables, the chunks are added to cleared tables by atomics, or the slots are: atomics_pay.)
// ---------------------------------------------------------------------------------------------
constexpr int kCoocTokens = 128;     // tokens per tile: four k-steps of the 32x32x32 int8 MFMA
constexpr int kCoocStride = 144;     // bytes per tile row: 128 tokens + 16, which spreads 32 rows over all banks
constexpr int kCoocGroups = 64;      // rows of the group tile
constexpr int kCoocChunksMax = 16;   // partial tables per cut
constexpr int kCoocChunkTokensMax = 32640;   // a chunk's counts are stored as 16-bit values
constexpr int kCoocMaxE = 512;
constexpr int kCoocPartMaxE = 256;   // experts up to which the workspace holds partial tables
constexpr int kCoocStaged = 8192;    // slots worked out together (32 KiB of LDS): a lane per token of eight
constexpr int kCoocAddedGroups = 256;   // workgroups aimed at where chunks are added up (512: E = 320, 4,096 tokens 33 -> 39 us)
constexpr int kCoocOwnK = 8;         // most slots of a token that the matrix kernel works out itself

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef i32x4 i32x4_align4 __attribute__((aligned(4)));
typedef int32_t i32x16 __attribute__((ext_vector_type(16)));

struct CoocParams {
  const int32_t *ids;
  const int32_t *expert_to_rank;
  int32_t T, K, E, G;
  int32_t sub_log2;            // places per token: 2^sub_log2 >= K
  int32_t ncuts;
  int32_t chunks;              // gridDim.x of the matrix kernel
  int32_t tokens_per_chunk;    // a multiple of kCoocTokens
  int32_t added;               // the tables are added to C, CG and base instead of stored as parts
  int32_t ng[kMaxCuts], per[kMaxCuts];
  uint8_t *slot_bits;          // [T * K]: bit 0 first valid occurrence, bit 1 + c alone in its group under cut c
  uint16_t *part[kMaxCuts];    // [chunks][E*E + E*ng + 64 (+1)]: C, CG and base of one chunk; a chunk has < 2^15 tokens
  int32_t *C[kMaxCuts], *CG[kMaxCuts], *base[kMaxCuts];
  int32_t *status;
};

__host__ __device__ static inline int64_t cooc_part_ints(int64_t E, int64_t ng) { return E * E + E * ng + 64; }   // values per chunk
__host__ __device__ static inline int64_t cooc_part_words(int64_t E, int64_t ng) { return (cooc_part_ints(E, ng) + 1) / 2; }   // 32-bit words they take

// One lane per routing slot (K > 8); the K slots of a token sit in 2^sub_log2 consecutive lanes and
// learn about each other through shuffles, eight in flight at a time.
__global__ __launch_bounds__(kSwapThreads) void swap_slots_kernel(CoocParams p) {
  const int sub = 1 << p.sub_log2;
  const int lane = lane_id();
  const int k = lane & (sub - 1);
  const int sub0 = lane & ~(sub - 1);
  const int64_t t = ((int64_t)blockIdx.x * kSwapThreads + threadIdx.x) >> p.sub_log2;
  const bool live = t < p.T && k < p.K;
  int a = -1, r = -1;   // my expert and its rank; -1 when the slot is empty, dropped or invalid
  if (live) {
    const int id = p.ids[t * p.K + k];
    const int rk = rank_of(p.expert_to_rank, p.E, p.G, id);
    if (rk == -1) flag(p.status, HM_ERR_BAD_ID);
    if (rk >= 0) {
      a = id;
      r = rk;
    }
  }
  bool first = a >= 0;   // the selected experts form a set: the first occurrence stands for it
  for (int k0 = 0; k0 < p.K; k0 += 8) {
    int a1[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) a1[j] = __shfl(a, sub0 + ((k0 + j) & (sub - 1)), kWave);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (k0 + j < k && a1[j] == a) first = false;
  }
  // The group of my rank under each cut, one byte per cut; equal bytes of two such words are counted
  // four cuts at a time (a zero byte of the exclusive or, found without a carry between bytes).
  __shared__ uint32_t groups_of_rank[kWave];
  if (threadIdx.x < kWave) {
    uint32_t packed = 0;
#pragma unroll
    for (int c = 0; c < kMaxCuts; ++c) packed |= (uint32_t)(threadIdx.x / p.per[c]) << (8 * c);
    groups_of_rank[threadIdx.x] = packed;
  }
  __syncthreads();
  const uint32_t pg = r >= 0 ? groups_of_rank[r] : 0u;
  const uint32_t mine = first ? pg : 0xFFFFFFFFu;   // no group has the number 255
  uint32_t in_group = 0;   // distinct selected experts in my expert's group, one byte per cut (at most 64)
  for (int k0 = 0; k0 < p.K; k0 += 8) {
    uint32_t g1[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) g1[j] = (uint32_t)__shfl((int)mine, sub0 + ((k0 + j) & (sub - 1)), kWave);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t x = g1[j] ^ pg;
      const uint32_t nonzero = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
      if (k0 + j < p.K) in_group += (nonzero ^ 0x80808080u) >> 7;
    }
  }
  if (live) {
    int bits = 0;
    if (first) {
      bits = 1;
#pragma unroll
      for (int c = 0; c < kMaxCuts; ++c)
        if (c < p.ncuts && ((in_group >> (8 * c)) & 0xFFu) == 1u) bits |= 2 << c;
    }
    p.slot_bits[t * p.K + k] = (uint8_t)bits;
  }
}

// D += A B for one 32x32 tile over 32 tokens; a lane's operand: 16 token bytes of row (lane % 32).
__device__ __forceinline__ i32x16 mfma_i8(i32x4 a, i32x4 b, i32x16 acc) {
  return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
}

// What a slot marks in the tiles: its expert, the expert's group, whether it is alone there; 0 if it marks nothing (no valid
// expert, or not the first with it in its token).
constexpr uint32_t kMarks = 1u << 31, kAlone = 1u << 15;
__device__ __forceinline__ uint32_t mark_of(int expert, uint32_t group, bool alone) {
  return kMarks | group << 16 | (alone ? kAlone : 0u) | (uint32_t)expert;
}

// The marks of a token of up to eight slots, by the one lane that holds it.  Groups are bits of BITS: one that has been seen
// twice, copies of an expert aside, is nobody's alone.  (A lane per slot that compares itself with the others
// took four times the instructions for a token, and the workgroups of all cuts and panels repeat them: 6.5 us for the 1,024
// tokens of a chunk on one CU.)
template <typename BITS>
__device__ __forceinline__ void mark_token(const int (&id)[kCoocOwnK], int E, const uint8_t *group_of, bool &bad, uint32_t (&mark)[kCoocOwnK]) {
  uint32_t expert[kCoocOwnK], group[kCoocOwnK];
  BITS once = 0, twice = 0;
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) {
    group[k] = group_of[min((uint32_t)id[k] + 1u, (uint32_t)E + 1u)];   // entry 0: id -1, E + 1: out of range
    bad = bad || group[k] == 0xFEu;
    expert[k] = group[k] < kWave ? (uint32_t)id[k] : 0x10000u + k;   // equal to no other
  }
  __builtin_amdgcn_sched_barrier(0);   // here and below: all comparisons at once would need more registers than there are
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) {
    uint32_t same = 1;   // 0 if an earlier slot has the expert
#pragma unroll
    for (int j = 0; j < k; ++j) same = min(same, expert[j] ^ expert[k]);
    const bool first = same != 0 && group[k] < kWave;
    const BITS bit = first ? (BITS)1 << group[k] : (BITS)0;
    mark[k] = first ? expert[k] | group[k] << 16 | kMarks : 0u;
    twice |= once & bit;
    once |= bit;
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k)
    if (mark[k] && !((twice >> group[k]) & 1)) mark[k] |= kAlone;
}

// A lane's column of a 32x32 tile, rows 8 (r / 4) + r % 4 from element `at` on, as far as they are below `rows`.
__device__ __forceinline__ void store_tile(uint16_t *part, const i32x16 &acc, int at, int width, int rows) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (8 * (r / 4) + r % 4 < rows) part[at + (8 * (r / 4) + r % 4) * width] = (uint16_t)acc[r];
}
__device__ __forceinline__ void add_tile(int32_t *table, const i32x16 &acc, int at, int width, int rows) {
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (8 * (r / 4) + r % 4 < rows && acc[r]) atomicAdd(&table[at + (8 * (r / 4) + r % 4) * width], acc[r]);
}

// Workgroup (chunk, cut, panel of 32 or 64 columns of C); the first waves hold one 32x32 tile of C each.  A workgroup
// needs the S tile of its own columns only; the panels repeat the marks of the chunk's slots and the A tile.  All
// sixteen waves mark.  One column of tiles up to 128 experts, so that four cuts and sixteen chunks are a workgroup per
// CU, two for 256 (E = 256, four cuts, the whole call: 8,192 tokens 33.7 us with one, 28.1 with two, 65,536 92 and 58).
// The whole call, graphs of ten, four cuts, K = 8, with a lane per slot and panels of 64 and 128 columns -> now, us: E = 128 1,024
// tokens 19.8 -> 14.6, 16,384 26.6 -> 21.1, 65,536 48.3 -> 40.2; E = 256 1,024 23.7 -> 21.2, 8,192 30.7 -> 27.7, 65,536 64.5 -> 57.4; by
// atomics per slot -> now: E = 320 4,096 77 -> 33, 30,000 131 -> 74, E = 512 (64 ranks, Zipf) 4,096 339 -> 54, 30,000 1,622 -> 124.
// Loops stay loops: unrolled, they cost the registers of the accumulators, which then live in memory.
//
// Per tile: mark | barrier | multiply | barrier.  Nothing waits for a tile to be cleared: with one column of tiles the rows of A
// are read by one wave, which clears them behind its reads; with two, the lanes that marked them clear them (a
// token's places belong to one wave, so it may mark the next tile without a barrier), or, for K > 8, whose tokens are
// spread over waves, all of them clear A behind a third barrier.  S and M, which several
// waves read, are there twice, and the one not in use is cleared while the other is multiplied.
constexpr int kCoocThreads = 1024;
constexpr int kCoocWaves = kCoocThreads / kWave;
constexpr int cooc_cols(int ne) { return ne == 8 ? 2 : 1; }   // tile columns of a panel
template <int NE, bool OWN_SLOTS>   // experts padded to 32 * NE
__global__ __launch_bounds__(kCoocThreads) void swap_cooc_kernel(CoocParams p) {
  constexpr int COLS = cooc_cols(NE), kCoocPanel = 32 * COLS;
  constexpr int kRows = kCoocPanel + kCoocGroups;   // of S and M
  constexpr int kVecs = (32 * NE + 2 * kRows) * kCoocStride / 16;
  constexpr int kRowVecs = kCoocTokens / 16;        // of a row without its pad, which nothing marks: a vector per lane clears S and M
  extern __shared__ __align__(16) uint8_t tiles[];
  uint8_t *const a_tile = tiles;                                   // [32 NE][stride]     A
  uint8_t *const sm_tiles = a_tile + 32 * NE * kCoocStride;        // twice [panel][stride] S, its experts, [64][stride] M
  uint32_t *const staged = (uint32_t *)(sm_tiles + 2 * kRows * kCoocStride);   // [tokens of a stage][2^sub_log2] marks
  __shared__ uint8_t group_of[32 * NE + 2];   // of expert e at e + 1; 0xFF none, 0xFE an error

  const int cut = blockIdx.y, panel = blockIdx.z;
  const int ng = p.ng[cut], per = p.per[cut];
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const i32x4 zero = {0, 0, 0, 0};
#pragma unroll 1
  for (int i = tid; i < kVecs; i += kCoocThreads) ((i32x4 *)tiles)[i] = zero;
  {
    const uint32_t per_recip16 = (65536u + (uint32_t)per - 1u) / (uint32_t)per;   // exact for ranks (below 64)
#pragma unroll 1
    for (int e = tid; e < p.E + 2; e += kCoocThreads) {
      const int r = e >= 1 && e <= p.E ? p.expert_to_rank[e - 1] : -1;
      group_of[e] = (uint8_t)(e == 0 ? 0xFFu : (unsigned)r < (unsigned)p.G ? ((uint32_t)r * per_recip16) >> 16 : 0xFEu);
    }
  }
  __syncthreads();

  // A token's marks lie in 2^sub_log2 places where a lane works a token out, one after the other where they are read: with places
  // padded to a power of two too, a tile of 33 slots cost twice the turns (E = 256, 40,000 tokens, four cuts: 165 us, now 128).
  const int sub_log2 = p.sub_log2, sub = 1 << sub_log2;
  const int per_token = OWN_SLOTS ? sub : p.K, places = kCoocTokens * per_token;   // of a tile
  const int stage_tokens = OWN_SLOTS ? kCoocStaged >> sub_log2 : kCoocStaged / places * kCoocTokens;   // 128 at least
  const uint32_t k_recip20 = ((1u << 20) + (uint32_t)p.K - 1u) / (uint32_t)p.K;   // exact below 8,192 for K <= 64
  const int64_t t_begin = (int64_t)blockIdx.x * p.tokens_per_chunk;
  const int64_t t_end = min((int64_t)p.T, t_begin + p.tokens_per_chunk);

  // What this wave accumulates: one tile of C, and from the last wave down at most one tile of this panel's CG.
  const int c_row = w / COLS, c_col = w % COLS;
  const bool has_c = c_row < NE && c_row < (p.E + 31) / 32;
  const int g_tiles = (ng + 31) / 32, g_job = kCoocWaves - 1 - w, g_row = g_job / g_tiles, g_col = g_job % g_tiles;
  const bool has_g = g_row < COLS;
  const bool counts_base = panel == 0 && w == kCoocWaves / 2;   // lane g: tokens of this chunk that touch group g
  constexpr bool kEither = NE * COLS + 4 <= kCoocWaves;   // no wave has both
  i32x16 acc, second;
  i32x16 &acc_g = kEither ? acc : second;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = second[r] = 0;
  int my_base = 0;
  const int op_at = (lane & 31) * kCoocStride + (lane >> 5) * 16;
  uint8_t *const c_a = a_tile + 32 * (has_c ? c_row : 0) * kCoocStride + op_at;
  const int c_s = 32 * c_col * kCoocStride + op_at, g_s = 32 * (has_g ? g_row : 0) * kCoocStride + op_at;
  const int g_m = (kCoocPanel + 32 * g_col) * kCoocStride + op_at;

  bool bad = false;
  uint8_t *sm = sm_tiles, *sm_next = sm_tiles + kRows * kCoocStride;
#pragma unroll 1
  for (int64_t stage0 = t_begin; stage0 < t_end; stage0 += stage_tokens) {
    const int tokens = (int)min((int64_t)stage_tokens, t_end - stage0);
    const int last = (tokens + kCoocTokens - 1) / kCoocTokens * places;   // places of the tiles to come
    if (OWN_SLOTS) {
#pragma unroll 1
      for (int t = tid; t < (last >> sub_log2); t += kCoocThreads) {
        int id[kCoocOwnK];
        uint32_t m[kCoocOwnK];
#pragma unroll
        for (int k = 0; k < kCoocOwnK; ++k) id[k] = -1;
        if (t < tokens) load_ids(p.ids + (stage0 + t) * p.K, p.K, 0, id);
        if (ng <= 32) mark_token<uint32_t>(id, p.E, group_of, bad, m);
        else mark_token<uint64_t>(id, p.E, group_of, bad, m);
        if (sub == kCoocOwnK) {
          *(i32x4 *)(staged + t * kCoocOwnK) = i32x4{(int)m[0], (int)m[1], (int)m[2], (int)m[3]};
          *(i32x4 *)(staged + t * kCoocOwnK + 4) = i32x4{(int)m[4], (int)m[5], (int)m[6], (int)m[7]};
        } else {
#pragma unroll
          for (int k = 0; k < kCoocOwnK / 2; ++k)
            if (k < sub) staged[(t << sub_log2) + k] = m[k];
        }
      }
    } else {
      constexpr int kAhead = 8;   // loads of a lane in flight together
      const int slots = tokens * p.K;
      const int32_t *const ids = p.ids + stage0 * p.K;
      const uint8_t *const slot_bits = p.slot_bits + stage0 * p.K;
#pragma unroll 1
      for (int i0 = tid; i0 < last; i0 += kAhead * kCoocThreads) {
        int id[kAhead], bits[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
          const int i = min(i0 + j * kCoocThreads, slots - 1);
          id[j] = ids[i];
          bits[j] = slot_bits[i];
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
          const int i = i0 + j * kCoocThreads;
          const uint32_t group = group_of[min((uint32_t)id[j] + 1u, (uint32_t)p.E + 1u)];
          const uint32_t m = mark_of(id[j], group, (bits[j] >> (1 + cut)) & 1);
          if (i < last) staged[i] = i < slots && (bits[j] & 1) ? m : 0u;
        }
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int first_place = 0; first_place < last; first_place += places) {
      int wrote = -1;   // where in A this lane's mark went
#pragma unroll 1
      for (int i = tid; i < places; i += kCoocThreads) {
        const uint32_t m = staged[first_place + i];
        if (!(m & kMarks)) continue;
        const int token = OWN_SLOTS ? i >> sub_log2 : (int)((uint32_t)i * k_recip20 >> 20);
        const int expert = (int)(m & 0x1FFu), column = expert - kCoocPanel * panel;
        if (m & kAlone) {
          const int at = expert * kCoocStride + token;
          a_tile[at] = 1;
          if (OWN_SLOTS) wrote = at;
        }
        if ((unsigned)column < (unsigned)kCoocPanel) sm[column * kCoocStride + token] = 1;
        sm[(kCoocPanel + (m >> 16 & 0x3Fu)) * kCoocStride + token] = 1;
      }
      __syncthreads();
      if (has_c) {
        i32x4 a_op[kCoocTokens / 32], s_op[kCoocTokens / 32];
#pragma unroll
        for (int step = 0; step < kCoocTokens / 32; ++step) {
          a_op[step] = *(const i32x4 *)(c_a + 32 * step);
          s_op[step] = *(const i32x4 *)(sm + c_s + 32 * step);
        }
        if (COLS == 1) {
#pragma unroll
          for (int step = 0; step < kCoocTokens / 32; ++step) *(i32x4 *)(c_a + 32 * step) = zero;
        }
#pragma unroll
        for (int step = 0; step < kCoocTokens / 32; ++step) acc = mfma_i8(a_op[step], s_op[step], acc);
      }
      if (has_g) {
#pragma unroll
        for (int step = 0; step < kCoocTokens / 32; ++step)
          acc_g = mfma_i8(*(const i32x4 *)(sm + g_s + 32 * step), *(const i32x4 *)(sm + g_m + 32 * step), acc_g);
      }
      if (counts_base) {   // bytes are 0 / 1, so a word's population count is its number of tokens
        const i32x4 *row = (const i32x4 *)(sm + (kCoocPanel + lane) * kCoocStride);
#pragma unroll
        for (int i = 0; i < kCoocTokens / 16; ++i) {
          const i32x4 v = row[i];
          my_base += __popc(v[0]) + __popc(v[1]) + __popc(v[2]) + __popc(v[3]);
        }
      }
#pragma unroll 1
      for (int i = tid; i < kRows * kRowVecs; i += kCoocThreads) ((i32x4 *)(sm_next + i / kRowVecs * kCoocStride))[i % kRowVecs] = zero;
      uint8_t *const used = sm;
      sm = sm_next;
      sm_next = used;
      __syncthreads();
      if (COLS > 1) {   // two waves read a row of A
        if (OWN_SLOTS) {   // a lane has one place of a tile: it clears what it marked
          if (wrote >= 0) a_tile[wrote] = 0;
        } else {   // the slots of a token are spread over waves
#pragma unroll 1
          for (int i = tid; i < 32 * NE * kRowVecs; i += kCoocThreads) ((i32x4 *)(a_tile + i / kRowVecs * kCoocStride))[i % kRowVecs] = zero;
          __syncthreads();
        }
      }
    }
  }
  if (OWN_SLOTS && bad && cut == 0 && panel == 0) flag(p.status, HM_ERR_BAD_ID);

  // Accumulator layout of a 32x32 tile: register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4,
  // column l % 32.
  const int64_t cg_at = (int64_t)p.E * p.E, base_at = cg_at + (int64_t)p.E * ng;
  uint16_t *const part = p.part[cut] + (int64_t)blockIdx.x * 2 * cooc_part_words(p.E, ng);
  const int col = lane & 31, row_hi = (lane >> 5) * 4;
  if (has_c && kCoocPanel * panel + 32 * c_col + col < p.E) {
    const int a0 = 32 * c_row + row_hi, at = a0 * p.E + kCoocPanel * panel + 32 * c_col + col;   // E <= 512
    if (!p.added) store_tile(part, acc, at, p.E, p.E - a0);
    else add_tile(p.C[cut], acc, at, p.E, p.E - a0);
  }
  if (has_g && 32 * g_col + col < ng) {
    const int a0 = kCoocPanel * panel + 32 * g_row + row_hi, at = a0 * ng + 32 * g_col + col;
    if (!p.added) store_tile(part + cg_at, acc_g, at, ng, p.E - a0);
    else add_tile(p.CG[cut], acc_g, at, ng, p.E - a0);
  }
  if (counts_base) {
    if (!p.added) part[base_at + lane] = (uint16_t)my_base;
    else if (my_base) atomicAdd(&p.base[cut][lane], my_base);
  }
}

// Sums the chunks' partial tables into the tables swap_build_kernel reads; blockIdx.y is the cut and
// blockIdx.x a 32 x 32 tile of C, then of CG.  A lane sums four neighbouring values, all chunks' loads in
// flight, and the tile is turned round in LDS, so that the transposes are written in whole lines too (one lane per
// value wrote them a word per line: kernel trace 6.6 us for 128 experts and four cuts, 9.2 us for 256; now 4.7 and
// 6.2).  L is the diagonal of C and L0[a] the entry of CG in a's own group (every token that selects a
// selects something there), so neither needs a table of its own upstream.  Where the chunks were added up by atomics
// already (cp.added), the tables are read back for the transposes, L and L0.
constexpr int kTile = 32;
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef u16x4 u16x4_align2 __attribute__((aligned(2)));
__host__ __device__ static inline int reduce_tiles(int E, int ng) {
  const int rows = (E + kTile - 1) / kTile;
  return rows * (rows + (ng + kTile - 1) / kTile);
}
__global__ __launch_bounds__(kSwapThreads) void swap_reduce_kernel(SwapParams p, CoocParams cp) {
  __shared__ int32_t turned[kTile][kTile + 1];
  const int cut = blockIdx.y;
  const int E = p.E, ng = p.ng[cut];
  if ((int)blockIdx.x >= reduce_tiles(E, ng)) return;
  const int64_t stride = 2 * cooc_part_words(E, ng);   // 16-bit values per chunk
  const uint16_t *const part = cp.part[cut];
  const int tile_rows = (E + kTile - 1) / kTile;
  const bool of_c = (int)blockIdx.x < tile_rows * tile_rows;
  const int index = of_c ? (int)blockIdx.x : (int)blockIdx.x - tile_rows * tile_rows;
  const int tile_cols = of_c ? tile_rows : (ng + kTile - 1) / kTile, width = of_c ? E : ng;
  const int a0 = index / tile_cols * kTile, b0 = index % tile_cols * kTile;
  const int row = threadIdx.x >> 3, col = (threadIdx.x & 7) * 4;
  const int a = a0 + row, b = b0 + col;
  int sum[4] = {0, 0, 0, 0};
  if (a < E && b < width) {
    const uint16_t *at = part + (of_c ? 0 : (int64_t)E * E) + (int64_t)a * width + b;
    int32_t *const out = (of_c ? p.C[cut] : p.CG[cut]) + (int64_t)a * width + b;
    if (cp.added) {
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] = b + e < width ? out[e] : 0;
    } else if (b + 4 <= width) {
      u16x4 v[kCoocChunksMax];   // every load unconditional (the last chunk again), so that none waits for another
#pragma unroll
      for (int c = 0; c < kCoocChunksMax; ++c) v[c] = *(const u16x4_align2 *)(at + min(c, cp.chunks - 1) * stride);
#pragma unroll
      for (int c = 0; c < kCoocChunksMax; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += c < cp.chunks ? v[c][e] : 0;
    } else {   // up to three values left: the last one again for what is missing, for the same reason
      uint16_t v[kCoocChunksMax][3];
#pragma unroll
      for (int c = 0; c < kCoocChunksMax; ++c)
#pragma unroll
        for (int e = 0; e < 3; ++e) v[c][e] = at[min(c, cp.chunks - 1) * stride + min(e, width - 1 - b)];
#pragma unroll
      for (int c = 0; c < kCoocChunksMax; ++c)
#pragma unroll
        for (int e = 0; e < 3; ++e) sum[e] += c < cp.chunks && b + e < width ? v[c][e] : 0;
    }
    const int rank = p.expert_to_rank[a];
    const bool placed = (unsigned)rank < (unsigned)p.G;
    const int own = of_c ? a : placed ? rank / p.per[cut] : 0;   // the column L or L0 is taken from
    if (cp.added) {
    } else if (b + 4 <= width) {
      *(i32x4_align4 *)out = (i32x4){sum[0], sum[1], sum[2], sum[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (b + e < width) out[e] = sum[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (b + e == own) {
        if (of_c) p.L[cut][a] = sum[e];
        else if (cut == 0) p.L0[a] = placed ? sum[e] : 0;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) turned[row][col + e] = sum[e];
  __syncthreads();
  const int b_out = b0 + row, a_out = a0 + col;   // a row of the transpose
  if (b_out < width && a_out < E && (of_c || p.cg_by_group[cut])) {
    int32_t *const out = (of_c ? p.CT[cut] : p.CGT[cut]) + (int64_t)b_out * E + a_out;
    if (a_out + 4 <= E) {
      *(i32x4_align4 *)out = (i32x4){turned[col][row], turned[col + 1][row], turned[col + 2][row], turned[col + 3][row]};
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (a_out + e < E) out[e] = turned[col + e][row];
    }
  }
  if (!cp.added && blockIdx.x == 0 && threadIdx.x < kWave) {
    const uint16_t *at = part + (int64_t)E * E + (int64_t)E * ng + threadIdx.x;
    int v[kCoocChunksMax], base = 0;
#pragma unroll
    for (int c = 0; c < kCoocChunksMax; ++c) v[c] = at[min(c, cp.chunks - 1) * stride];
#pragma unroll
    for (int c = 0; c < kCoocChunksMax; ++c) base += c < cp.chunks ? v[c] : 0;
    p.base[cut][threadIdx.x] = base;
  }
}

// One lane per (c, j) of a cut and kBuildRows row experts r: blockIdx.y is the block of rows and
// blockIdx.x runs over the column blocks (256 consecutive (c, j)) of all cuts, one cut after the
// other.  The loads of all rows are issued before the first value is put together, so a lane
// waits for memory once, and the waves are long enough for the chip not to be bound by starting
// them.  The two divisions a lane needs are multiplications by rounded-up reciprocals: c = l / ng
// (exact for l < 2^32 / ng, and l < 64 E < 2^19) and group = rank / per (rank < 64).
constexpr int kBuildRows = 4;

// The same for cuts of a multiple of four groups, where a lane takes four neighbouring groups j of its c:
// their unswapped counts are read once for all rows, a row costs one 16-byte store, and only the lanes
// that hold the group of c or of r look anything up (a quarter of the lanes, each of whose rows is
// a few instructions: 256 experts, four cuts, 15.7 MB of Z, kernel trace 12.8 -> 9.3 us, where the fastest launches take 7.5).
__device__ __forceinline__ void build_quads(const SwapParams &p, int cut, int l, int r0) {
  const int ng = p.ng[cut], nq = ng / 4;
  const int32_t *__restrict__ const C = p.C[cut];
  const int32_t *__restrict__ const CT = p.CT[cut];
  const int32_t *__restrict__ const CG = p.CG[cut];
  const int32_t *__restrict__ const CGT = p.CGT[cut];
  const int by_group = p.cg_by_group[cut];
  const int32_t *__restrict__ const L = p.L[cut];
  const int32_t *__restrict__ const L0 = p.L0;
  const unsigned per_reciprocal = p.per_reciprocal[cut];
  const int c = nq == 1 ? l : (int)__umulhi((unsigned)l, p.quad_reciprocal[cut]);
  const int jq = l - c * nq;
  const int rk = p.expert_to_rank[c];
  const bool c_ok = (unsigned)rk < (unsigned)p.G;
  const int gc = !c_ok ? -1 : per_reciprocal ? (int)__umulhi((unsigned)rk, per_reciprocal) : rk;
  const i32x4 base = *(const i32x4_align4 *)(p.base[cut] + 4 * jq);
  const int L_c = L[c], L0_c = L0[c];
  const bool holds_c = c_ok && (gc >> 2) == jq;
  int group_r[kBuildRows];   // r's group if it is one of the four and not c's
  int cg[kBuildRows], ct[kBuildRows], cgt[kBuildRows], cc[kBuildRows], L_r[kBuildRows], L0_r[kBuildRows];
  bool gains[kBuildRows], bad = false;
#pragma unroll
  for (int i = 0; i < kBuildRows; ++i) {
    const int r = min(r0 + i, p.E - 1);   // uniform
    const int rr = p.expert_to_rank[r];
    const bool r_ok = (unsigned)rr < (unsigned)p.G;
    const int gr = !r_ok ? -1 : per_reciprocal ? (int)__umulhi((unsigned)rr, per_reciprocal) : rr;
    bad = bad || !r_ok || !c_ok;
    const bool moves = r_ok && c_ok && gr != gc;
    gains[i] = moves && holds_c;
    group_r[i] = moves && (gr >> 2) == jq ? gr & 3 : -1;
    cg[i] = ct[i] = cgt[i] = cc[i] = 0;
    L_r[i] = L[r];
    L0_r[i] = L0[r];
    if (gains[i]) {
      cg[i] = CG[(int64_t)r * ng + gc];
      ct[i] = CT[(int64_t)r * p.E + c];
    }
    if (group_r[i] >= 0) {
      cgt[i] = CGT[by_group ? gr * p.E + c : c * ng + gr];
      cc[i] = C[(int64_t)r * p.E + c];
    }
  }
  if (bad && jq == 0) flag(p.status, HM_ERR_BAD_ID);
#pragma unroll
  for (int i = 0; i < kBuildRows; ++i) {
    i32x4 z = base;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      z[e] += gains[i] && (gc & 3) == e ? (L0_r[i] - cg[i]) - (L_c - ct[i]) : 0;
      z[e] += group_r[i] == e ? (L0_c - cgt[i]) - (L_r[i] - cc[i]) : 0;
    }
    if (r0 + i < p.E) *(i32x4_align4 *)(p.Z[cut] + ((int64_t)(r0 + i) * p.E * ng + 4 * (int64_t)l)) = z;
  }
}

// QUADS: whether any cut takes four groups per lane; the registers that takes slow the other form down (E = 300 through
// the atomics, four cuts, 1,024 tokens, K = 2, the whole call: 56.8 -> 55.3 us).
template <bool QUADS>
__global__ __launch_bounds__(kSwapThreads) void swap_build_kernel(SwapParams p) {
  int cut = 0, block = blockIdx.x;
  while (cut + 1 < p.ncuts && block >= p.build_blocks[cut]) block -= p.build_blocks[cut++];
  const int ng = p.ng[cut], r0 = blockIdx.y * kBuildRows;
  const int l = block * kSwapThreads + threadIdx.x;
  if (QUADS && p.quads[cut]) {
    if (l < p.E * (ng / 4)) build_quads(p, cut, l, r0);
    return;
  }
  if (l >= p.E * ng) return;
  const int32_t *__restrict__ const C = p.C[cut];
  const int32_t *__restrict__ const CT = p.CT[cut];
  const int32_t *__restrict__ const CG = p.CG[cut];
  const int32_t *__restrict__ const CGT = p.CGT[cut];
  const int32_t *__restrict__ const L = p.L[cut];
  const int32_t *__restrict__ const L0 = p.L0;
  int32_t *__restrict__ const Z = p.Z[cut];
  const unsigned per_reciprocal = p.per_reciprocal[cut];
  const int c = ng == 1 ? l : (int)__umulhi((unsigned)l, p.ng_reciprocal[cut]);
  const int j = l - c * ng;
  const int rk = p.expert_to_rank[c];
  const bool c_ok = (unsigned)rk < (unsigned)p.G;
  const int gc = !c_ok ? -1 : per_reciprocal ? (int)__umulhi((unsigned)rk, per_reciprocal) : rk;
  const int base = p.base[cut][j];
  int add[kBuildRows], sub_[kBuildRows];   // val = base + add - sub
  bool bad = false;
#pragma unroll
  for (int i = 0; i < kBuildRows; ++i) {
    const int r = min(r0 + i, p.E - 1);
    const int rr = p.expert_to_rank[r];
    const bool r_ok = (unsigned)rr < (unsigned)p.G;
    const int gr = !r_ok ? -1 : per_reciprocal ? (int)__umulhi((unsigned)rr, per_reciprocal) : rr;
    add[i] = sub_[i] = 0;
    if (!r_ok || !c_ok) {
      bad = true;
    } else if (gr != gc && (j == gc || j == gr)) {
      const int a = j == gc ? r : c, b = j == gc ? c : r;   // group j gains tokens of a, loses tokens of b
      int cba = 0, cg;
      if (p.transposed) {   // every read runs along row r of a table, or along c
        cba = j == gc ? CT[(int64_t)r * p.E + c] : C[(int64_t)r * p.E + c];
        cg = j == gc ? CG[(int64_t)r * ng + j] : CGT[p.cg_by_group[cut] ? j * p.E + c : c * ng + j];
      } else {
#pragma unroll 8
        for (int k = 0; k < p.copies; ++k) cba += C[((int64_t)k * p.E + b) * p.E + a];
        cg = CG[(int64_t)a * ng + j];
      }
      add[i] = L0[a] - cg;
      sub_[i] = L[b] - cba;
    }
  }
  if (bad && j == 0) flag(p.status, HM_ERR_BAD_ID);
#pragma unroll
  for (int i = 0; i < kBuildRows; ++i)
    if (r0 + i < p.E) Z[((int64_t)(r0 + i) * p.E) * ng + l] = base + (add[i] - sub_[i]);
}

// ---------------------------------------------------------------------------------------------
// selection
// ---------------------------------------------------------------------------------------------
constexpr int kMaxDim = 4;

struct SelectParams {
  int32_t d, G, E;
  int32_t U[kMaxDim];
  double M, v, gamma;
  const int32_t *z_inter[kMaxDim];
  const int32_t *z_intra;
  double scale_inter[kMaxDim], alpha_inter[kMaxDim], beta_inter[kMaxDim];
  double scale_intra, alpha_intra, beta_intra;
  double *Q;
  double *block_min;    // workspace [nblocks]
  int32_t *block_arg;   // workspace [nblocks]
  int32_t nblocks;
  int32_t *best_pair;
  double *best_time;
};

// x[0 .. N) of a term's counts, 0 beyond n <= N: all loads in flight together, and the counts stay in
// registers for the sum after the maximum (counts are >= 0, so the padding changes neither the maximum
// nor, skipped, the sum).
template <int N>
__device__ __forceinline__ void load_counts(const int32_t *x, int n, int (&v)[N]) {
  // every load unconditional (the last counts again beyond n), so that none waits for another
  if ((n & 3) == 0) {
#pragma unroll
    for (int j = 0; j < N; j += 4) {
      const i32x4 w = *(const i32x4_align4 *)(x + min(j, n - 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j + e] = w[e];
    }
  } else {
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = x[min(j, n - 1)];
  }
#pragma unroll
  for (int j = 0; j < N; ++j) v[j] = j < n ? v[j] : 0;
}

// The smooth maximum of Eq.(11) of n <= N counts.  Every lane is a chain of fp64 operations and there
// is about one wave per SIMD, so the chain is what counts: a whole gamma is raised for eight counts
// side by side, one pass over its bits for all of them; the sum itself stays in the order of the
// counts.
template <int N>
__device__ __forceinline__ double smooth_max(const int32_t *x, int n, double gamma) {
  int v[N];
  load_counts<N>(x, n, v);
  int mi = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) mi = max(mi, v[j]);
  const double m = (double)mi;
  if (gamma <= 0.0 || m == 0.0) return m;
  // A small whole gamma (the paper uses 10) needs no pow per entry: square-and-multiply gives the
  // same power to a few ulp, and a lane is otherwise a serial chain of up to 64 pow calls.
  const int whole = (gamma <= 64.0 && gamma == (double)(int)gamma) ? (int)gamma : 0;
  double sum = 0.0;
  if (whole) {
    const double inv_m = 1.0 / m;
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += 8) {
      if (i0 < n) {
        double acc[8], sq[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          sq[j] = (double)v[i0 + j] * inv_m;   // within an ulp of the quotient
          acc[j] = 1.0;
        }
        for (int e = whole;;) {
          if (e & 1) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] *= sq[j];
          }
          if ((e >>= 1) == 0) break;
#pragma unroll
          for (int j = 0; j < 8; ++j) sq[j] *= sq[j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (i0 + j < n) sum += acc[j];
      }
    }
  } else {
    for (int i = 0; i < n; ++i) sum += pow((double)x[i] / m, gamma);
  }
  return m * pow(sum, 1.0 / gamma);
}

__device__ __forceinline__ void keep_better(double &val, int32_t &arg, double v, int32_t a) {
  const bool better = a >= 0 && (arg < 0 || v < val || (v == val && a < arg));   // among equal times the lower pair index
  val = better ? v : val;
  arg = better ? a : arg;
}
__device__ __forceinline__ void wave_argmin(double &val, int32_t &arg) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) keep_better(val, arg, __shfl_xor(val, off, kWave), __shfl_xor(arg, off, kWave));
}

// Q of 64 pairs by a workgroup: a wave per term of Eq.(8) (the Inter levels 1 .. d-1, then the Intra
// level), a lane per pair, so that the waves with few groups are done early instead of waiting for the
// lanes of the widest cut, and everything about a term is uniform.  The terms are then added in the
// order of the levels, so Q has the bits of a serial evaluation.  Kernel trace, four terms: 128 experts
// 6.8 us, 256 experts 10.2 us (four lanes per pair side by side: 8.1 and 14.1).
template <int N>   // most groups of a term: 32 or 64
__global__ __launch_bounds__(kSelectThreads) void swap_q_kernel(SelectParams p) {
#pragma clang fp contract(off)
  __shared__ double s_term[kMaxDim][kSelectPairs];
  const int lane = lane_id();
  const int term = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int64_t rc = (int64_t)blockIdx.x * kSelectPairs + lane;
  const bool live = rc < (int64_t)p.E * p.E;
  if (term < p.d) {
    const bool intra = term == p.d - 1;
    const int i = intra ? 0 : term + 1;
    const int n = intra ? p.G : p.U[i];
    const int32_t *x = (intra ? p.z_intra : p.z_inter[i]) + (live ? rc : 0) * n;
    const double fan = intra ? (double)(p.G / p.U[p.d - 1]) : (double)(p.U[i] / p.U[intra ? 0 : i - 1]);
    const double scale = intra ? p.scale_intra : p.scale_inter[i];
    const double beta = intra ? p.beta_intra : p.beta_inter[i], alpha = intra ? p.alpha_intra : p.alpha_inter[i];
    const double volume = fan * scale * smooth_max<N>(x, n, p.gamma) * p.M * p.v;
    s_term[term][lane] = volume * beta + alpha;
  }
  __syncthreads();
  if (term != 0) return;
  double q = 0.0;
  for (int j = 0; j < p.d; ++j) q = q + s_term[j][lane];
  if (live) p.Q[rc] = q;
  int32_t arg = live ? (int32_t)rc : -1;
  wave_argmin(q, arg);
  if (lane == 0) {
    p.block_min[blockIdx.x] = q;
    p.block_arg[blockIdx.x] = arg;
  }
}

// The first of the smallest block minima.  One workgroup, bound by its trip to memory and the steps to
// one value: four minima per lane in flight, then shuffles within the waves and one step across them.
constexpr int kArgminThreads = 1024;
__global__ __launch_bounds__(kArgminThreads) void swap_argmin_kernel(SelectParams p) {
  __shared__ double s_val[kArgminThreads / kWave];
  __shared__ int32_t s_arg[kArgminThreads / kWave];
  double best = 0.0;
  int32_t arg = -1;
  for (int b0 = 0; b0 < p.nblocks; b0 += 4 * kArgminThreads) {
    double v[4];
    int32_t a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int b = b0 + j * kArgminThreads + (int)threadIdx.x;
      v[j] = b < p.nblocks ? p.block_min[b] : 0.0;
      a[j] = b < p.nblocks ? p.block_arg[b] : -1;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) keep_better(best, arg, v[j], a[j]);
  }
  wave_argmin(best, arg);
  if (lane_id() == 0) {
    s_val[threadIdx.x / kWave] = best;
    s_arg[threadIdx.x / kWave] = arg;
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  constexpr int kWaves = kArgminThreads / kWave;
  best = s_val[threadIdx.x & (kWaves - 1)];
  arg = s_arg[threadIdx.x & (kWaves - 1)];
  wave_argmin(best, arg);
  if (threadIdx.x == 0) {
    p.best_pair[0] = arg / p.E;
    p.best_pair[1] = arg % p.E;
    *p.best_time = best;
  }
}

// The chosen swap (Section IV): the two placement entries trade places; the diagonal (no swap won
// Eq.(10)) and out-of-range indices change nothing.
__global__ void swap_apply_kernel(int32_t *__restrict__ expert_to_rank, int32_t E, const int32_t *__restrict__ pair) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const int32_t r = pair[0], c = pair[1];
  if (r < 0 || r >= E || c < 0 || c >= E || r == c) return;
  const int32_t g = expert_to_rank[r];
  expert_to_rank[r] = expert_to_rank[c];
  expert_to_rank[c] = g;
}

// The co-occurrence kernel may use more dynamic LDS than a kernel gets by default (64 KiB); ask
// once.  False: the tables stay in global memory.
static bool swap_factors_lds_ready() {
  static const bool ok = [] {
    const hipError_t e = hipFuncSetAttribute((const void *)swap_factors_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             kSwapLds * (int)sizeof(int32_t));
    if (e != hipSuccess) (void)hipGetLastError();   // not sticky: do not let it fail the next launch check
    return e == hipSuccess;
  }();
  return ok;
}

// Private copies of C on the path with atomics: as many as fit 2 MiB per cut, at most
// kSwapCopiesMax (32 for E <= 128, 8 for E = 256): more copies spread the atomics of popular pairs,
// but each is cleared and summed again.  The matrix path keeps one summed C.
// Whether the workspace has partial tables of chunks (and a byte per slot): E <= 256 and chunks short enough for
// 16-bit counts.
static inline bool swap_has_parts(int64_t E, int64_t T) { return E <= kCoocPartMaxE && T <= (int64_t)kCoocChunksMax * kCoocChunkTokensMax; }
static inline int64_t swap_copies(int64_t E, int64_t T) {
  if (swap_has_parts(E, T)) return 1;
  int64_t n = kSwapCopiesMax;   // a power of two, so that a workgroup finds its copy with a mask
  while (n > 1 && n * E * E > (int64_t)(1 << 19)) n /= 2;
  return n;
}

// Workspace, in ints: L0 [E], then per cut base [64] | L [E] | CG [E * ng] | C [copies * E * E], and on the
// matrix path the partial tables of kCoocChunksMax chunks and the transposes of C and CG after that.
static inline int64_t swap_cut_ints(int64_t E, int64_t ng, int64_t T) {
  return 64 + E + E * ng + swap_copies(E, T) * E * E +
         (swap_has_parts(E, T) ? kCoocChunksMax * cooc_part_words(E, ng) + E * E + E * ng : 0);
}
// ... and, on the matrix path, one byte per routing slot at the very end.
static inline int64_t swap_slot_ints(int64_t T, int64_t K, int64_t E) { return swap_has_parts(E, T) ? (T * K + 3) / 4 : 0; }

// The matrix kernel for E experts and K slots, the columns of a panel and the dynamic LDS (0: the device does not grant that much).
typedef void (*cooc_kernel_t)(CoocParams);
struct CoocLaunch {
  cooc_kernel_t kernel;
  int ne, panel;
  size_t lds;
};
template <int NE, bool OWN_SLOTS>
static CoocLaunch cooc_launch() {
  constexpr size_t tiles = (size_t)(32 * NE + 2 * (32 * cooc_cols(NE) + kCoocGroups)) * kCoocStride, bytes = tiles + 4 * kCoocStaged;
  static const bool granted = [] {
    const hipError_t e = hipFuncSetAttribute((const void *)swap_cooc_kernel<NE, OWN_SLOTS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)bytes);
    if (e != hipSuccess) (void)hipGetLastError();   // not sticky: do not let it fail the next launch check
    return e == hipSuccess;
  }();
  return {swap_cooc_kernel<NE, OWN_SLOTS>, NE, 32 * cooc_cols(NE), granted ? bytes : 0};
}
template <bool OWN_SLOTS>
static CoocLaunch cooc_launch_for(int E) {
  return E <= 32    ? cooc_launch<1, OWN_SLOTS>()
         : E <= 64  ? cooc_launch<2, OWN_SLOTS>()
         : E <= 128 ? cooc_launch<4, OWN_SLOTS>()
         : E <= 256 ? cooc_launch<8, OWN_SLOTS>()
                    : cooc_launch<16, true>();   // there is no room for the bytes of swap_slots_kernel beyond
}

static inline int cooc_chunks(const CoocLaunch &cooc, bool parts, int64_t T, int64_t E, int ncuts) {
  const int64_t panels = (E + cooc.panel - 1) / cooc.panel, tiles = (T + kCoocTokens - 1) / kCoocTokens;
  const int64_t most = parts ? kCoocChunksMax : kCoocAddedGroups / (panels * ncuts), chunks = most > tiles ? tiles : most;
  return (int)(chunks < 1 ? 1 : chunks);
}

// Whether atomics per slot are faster than matrix products whose chunks are added up: with few slots per token or few groups, as
// the products take the same time however few marks a tile holds.  Two straight lines, us, through 4,701 shapes (256 < E <= 512, up to 520,000
// tokens; E <= 256, 522,241 to 800,000; one to eight slots, one to four cuts; ids drawn evenly): Z, the updates of C (a slot's K - 1
// others where it is alone in its group) and of L0, L and CG (in LDS or in memory), and the workgroups that put their tables
// together; against a time per tile of 128 tokens.  One or two tiles are matrices at any rate, but for next to no groups.  A popular few
// experts make only the atomics slower, so they have to be ahead by a fifth: of 4,105 shapes of more than two groups with even ids 277 lose
// more than 3 % by that (one half as much again) and 9 the other way round, of 2,980 with a Zipf router 71 and 131.
// Atomics / matrices: E = 512, cuts of 4 and 32, 65,536 tokens: K = 1 53 / 107, 2 63 / 110, 4 103 / 117 (Zipf 181 / 112), 8 (30,000
// tokens) 131 / 74; E = 260, 2, 4 and 8, 16,384 tokens: K = 1 24 / 34, 8 53 / 40; E = 256, 530,000 tokens: K = 1 46 / 145, 2 108 /
// 153, 3 220 / 157.
static bool atomics_pay(int64_t T, int64_t K, int64_t E, int ncuts, const int32_t *ng, bool in_lds, int ne, int chunks) {
  double groups = 0.0, others = 0.0, touched = 1.0;   // per slot: updates of C, words of L0, L and CG
  for (int c = 0; c < ncuts; ++c) {
    double alone = (double)(K - 1);
    for (int64_t k = 1; k < K; ++k) alone *= 1.0 - 1.0 / ng[c];
    groups += ng[c];
    others += alone;
    touched += 1.0 + (double)(K < ng[c] ? K : ng[c]);
  }
  const int64_t tiles = ((T + kCoocTokens - 1) / kCoocTokens + chunks - 1) / chunks;   // of a workgroup
  if (tiles <= 2 && groups > 4.0) return false;
  int64_t lanes = 1;
  while (lanes < K) lanes *= 2;
  const double pairs = (double)(E * E) * 1e-6, slots = (double)(T * K) * 1e-6, filled = (double)(T * lanes) / (256.0 * kFactorThreads);
  const double flush = filled < 1.0 ? filled : 1.0;   // of 256 workgroups
  const double atomics = in_lds ? 10.0 + 4.3 * pairs * groups + slots * (28.0 * others + 1.4 * touched) + 3.2 * ncuts + 6.6 * flush
                                : 45.0 + 2.4 * pairs * groups + 54.0 * slots * touched + 59.0 * flush;
  const double matrices = 15.0 + 6.0 * pairs * ncuts + 0.86 * pairs * groups + (double)tiles * (0.64 + 0.031 * (double)(ne + K));
  return 1.2 * atomics < matrices;
}

static inline bool swap_cuts_ok(int32_t G, int32_t ncuts, const int32_t *ng) {
  if (G < 1 || G > 64 || ncuts < 1 || ncuts > kMaxCuts || !ng) return false;
  for (int c = 0; c < ncuts; ++c)
    if (ng[c] < 1 || ng[c] > G || G % ng[c] != 0) return false;
  return true;
}

static hm_status swap_counts_launch(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K, int32_t E,
                                    int32_t G, int32_t ncuts, const int32_t *ng, int32_t *const *Z, int32_t *status,
                                    void *workspace, hipStream_t stream) {
  SwapParams p;
  p.ids = topk_ids;
  p.expert_to_rank = expert_to_rank;
  p.T = T;
  p.K = K;
  p.E = E;
  p.G = G;
  p.ncuts = ncuts;
  p.copies = (int32_t)swap_copies(E, T);
  p.sub = 1;
  while (p.sub < K) p.sub *= 2;
  p.ws = (int32_t *)workspace;
  p.L0 = p.ws;
  int64_t at = E, lds_at = E;
  for (int c = 0; c < kMaxCuts; ++c) {
    const int cc = c < ncuts ? c : 0;   // unused entries repeat cut 0 so that no pointer is left dangling
    p.ng[c] = ng[cc];
    p.per[c] = G / ng[cc];
    p.ng_reciprocal[c] = ng[cc] > 1 ? (uint32_t)((0x100000000ull + ng[cc] - 1) / ng[cc]) : 0u;
    p.per_reciprocal[c] = p.per[c] > 1 ? (uint32_t)((0x100000000ull + p.per[c] - 1) / p.per[c]) : 0u;
    p.Z[c] = Z[cc];
    if (c < ncuts) {
      p.base[c] = p.ws + at;
      p.L[c] = p.base[c] + 64;
      p.CG[c] = p.L[c] + E;
      p.C[c] = p.CG[c] + (int64_t)E * ng[c];
      at += swap_cut_ints(E, ng[c], T);
      p.lds_off[c] = (int32_t)lds_at;
      lds_at += (int64_t)E * (ng[c] + 1);
    } else {
      p.base[c] = p.base[0];
      p.L[c] = p.L[0];
      p.CG[c] = p.CG[0];
      p.C[c] = p.C[0];
      p.lds_off[c] = p.lds_off[0];
    }
  }
  p.status = status;
  // By matrices where there is room for the chunks' tables; beyond that (E > 256, or more than 522,240 tokens) the chunks
  // are added to cleared tables, as long as the marks of the slots need no room either and that is the faster way.
  const bool parts = swap_has_parts(E, T), own_slots = K <= kCoocOwnK;
  const bool in_lds = lds_at <= kSwapLds && swap_factors_lds_ready();
  CoocParams cp;
  cp.sub_log2 = 0;
  while ((1 << cp.sub_log2) < K) ++cp.sub_log2;
  CoocLaunch cooc = {nullptr, 0, 0, 0};
  if (parts || (own_slots && E <= kCoocMaxE)) cooc = own_slots ? cooc_launch_for<true>(E) : cooc_launch_for<false>(E);
  const int chunks = cooc.lds != 0 ? cooc_chunks(cooc, parts, T, E, ncuts) : 0;
  if (cooc.lds != 0 && (parts || !atomics_pay(T, K, E, ncuts, ng, in_lds, cooc.ne, chunks))) {
    p.ws_ints = parts ? 0 : at;   // parts are written in full by the kernels below: only the status word needs clearing
    p.use_lds = 0;
    p.transposed = 1;
    if (status || p.ws_ints) {
      const int64_t n = p.ws_ints > 0 ? p.ws_ints : 1;
      hipLaunchKernelGGL(swap_clear_kernel, dim3((unsigned)((n + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads), 0, stream, p);
      if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    }
    cp.ids = topk_ids;
    cp.expert_to_rank = expert_to_rank;
    cp.T = T;
    cp.K = K;
    cp.E = E;
    cp.G = G;
    cp.ncuts = ncuts;
    cp.added = parts ? 0 : 1;
    cp.slot_bits = (uint8_t *)(p.ws + at);
    const int panels = (E + cooc.panel - 1) / cooc.panel, tiles = (int)(((int64_t)T + kCoocTokens - 1) / kCoocTokens);
    cp.chunks = chunks;
    cp.tokens_per_chunk = (tiles + chunks - 1) / chunks * kCoocTokens;
    int max_tiles = 0;
    for (int c = 0; c < kMaxCuts; ++c) {
      const int64_t table = (int64_t)E * E, cg = (int64_t)E * p.ng[c];
      cp.ng[c] = p.ng[c];
      cp.per[c] = p.per[c];
      cp.C[c] = p.C[c];
      cp.CG[c] = p.CG[c];
      cp.base[c] = p.base[c];
      cp.part[c] = (uint16_t *)(p.C[c] + table);   // behind the summed C of the cut, and behind them the transposes;
      p.CT[c] = p.C[c] + table + (parts ? kCoocChunksMax * cooc_part_words(E, p.ng[c]) : 0);   // else they take copies of C
      p.cg_by_group[c] = parts || (p.copies - 2) * table >= cg;
      p.CGT[c] = p.cg_by_group[c] ? p.CT[c] + table : p.CG[c];
      if (c < ncuts && reduce_tiles(E, ng[c]) > max_tiles) max_tiles = reduce_tiles(E, ng[c]);
    }
    cp.status = status;
    if (T > 0 && !own_slots) {
      const int64_t lanes = (int64_t)T << cp.sub_log2;
      hipLaunchKernelGGL(swap_slots_kernel, dim3((unsigned)((lanes + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads), 0,
                         stream, cp);
      if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    }
    hipLaunchKernelGGL(cooc.kernel, dim3((unsigned)chunks, (unsigned)ncuts, (unsigned)panels), dim3(kCoocThreads), cooc.lds, stream, cp);
    if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    hipLaunchKernelGGL(swap_reduce_kernel, dim3((unsigned)max_tiles, (unsigned)ncuts), dim3(kSwapThreads), 0, stream, p, cp);
    if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  } else {
    p.transposed = 0;
    for (int c = 0; c < kMaxCuts; ++c) {
      p.CT[c] = p.CGT[c] = nullptr;
      p.cg_by_group[c] = 0;
    }
    p.ws_ints = at;
    p.use_lds = in_lds ? 1 : 0;
    hipLaunchKernelGGL(swap_clear_kernel, dim3((unsigned)((p.ws_ints + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads),
                       0, stream, p);
    if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    if (T > 0) {
      const int64_t tokens_per_block = (int64_t)(kFactorThreads / kWave) * (kWave / p.sub);
      int64_t blocks = ((int64_t)T + tokens_per_block - 1) / tokens_per_block;
      if (blocks > 256) blocks = 256;   // one per CU; every block flushes its LDS tables with atomics
      hipLaunchKernelGGL(swap_factors_kernel, dim3((unsigned)blocks), dim3(kFactorThreads),
                         p.use_lds ? (size_t)lds_at * sizeof(int32_t) : 0, stream, p);
      if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
    }
  }
  int64_t build_blocks = 0;
  bool any_quads = false;
  for (int c = 0; c < kMaxCuts; ++c) {
    p.quads[c] = p.transposed && p.ng[c] % 4 == 0 ? 1 : 0;
    p.quad_reciprocal[c] = p.quads[c] && p.ng[c] > 4 ? (uint32_t)((0x100000000ull + p.ng[c] / 4 - 1) / (p.ng[c] / 4)) : 0u;
    const int64_t lanes = (int64_t)E * (p.quads[c] ? p.ng[c] / 4 : p.ng[c]);
    p.build_blocks[c] = c < ncuts ? (int32_t)((lanes + kSwapThreads - 1) / kSwapThreads) : 0;
    build_blocks += p.build_blocks[c];
    any_quads = any_quads || (c < ncuts && p.quads[c]);
  }
  hipLaunchKernelGGL(any_quads ? swap_build_kernel<true> : swap_build_kernel<false>, dim3((unsigned)build_blocks, (unsigned)((E + kBuildRows - 1) / kBuildRows)),
                     dim3(kSwapThreads), 0, stream, p);
  return hm_launch_status();
}

}  // namespace hm

extern "C" size_t hm_swap_multi_workspace_bytes(int32_t T, int32_t K, int32_t E, int32_t G, int32_t ncuts, const int32_t *ng) {
  if (E < 1 || T < 0 || K < 1 || !hm::swap_cuts_ok(G, ncuts, ng)) return 0;
  int64_t ints = E + hm::swap_slot_ints(T, K, E);
  for (int c = 0; c < ncuts; ++c) ints += hm::swap_cut_ints(E, ng[c], T);
  return (size_t)ints * sizeof(int32_t);
}

extern "C" size_t hm_swap_workspace_bytes(int32_t T, int32_t K, int32_t E, int32_t ng) {
  if (E < 1 || T < 0 || K < 1 || ng < 1 || ng > 64) return 0;
  return (size_t)(E + hm::swap_cut_ints(E, ng, T) + hm::swap_slot_ints(T, K, E)) * sizeof(int32_t);
}

static hm_status swap_counts_checks(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K, int32_t E,
                                    const void *workspace) {
  if (!expert_to_rank || !workspace) return HM_ERR_NULL;
  hm_status st = hm_check_tk(T, K);
  if (st != HM_OK) return st;
  if (E < 1 || (int64_t)E * E * 64 > 2147483647LL) return HM_ERR_SHAPE;
  if (T > 0 && !topk_ids) return HM_ERR_NULL;
  return HM_OK;
}

extern "C" hm_status hm_swap_counts(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K,
                                    int32_t E, int32_t G, int32_t ng, int32_t *Z, int32_t *status, void *workspace,
                                    size_t workspace_bytes, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!Z) return HM_ERR_NULL;
  hm_status st = swap_counts_checks(topk_ids, expert_to_rank, T, K, E, workspace);
  if (st != HM_OK) return st;
  if (!hm::swap_cuts_ok(G, 1, &ng)) return HM_ERR_TOPOLOGY;
  if (workspace_bytes < hm_swap_workspace_bytes(T, K, E, ng)) return HM_ERR_WORKSPACE;
  return hm::swap_counts_launch(topk_ids, expert_to_rank, T, K, E, G, 1, &ng, &Z, status, workspace, (hipStream_t)hip_stream);
}

extern "C" hm_status hm_swap_counts_multi(const int32_t *topk_ids, const int32_t *expert_to_rank, int32_t T, int32_t K,
                                          int32_t E, int32_t G, int32_t ncuts, const int32_t *ng, int32_t *const *Z,
                                          int32_t *status, void *workspace, size_t workspace_bytes, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!Z || !ng) return HM_ERR_NULL;
  hm_status st = swap_counts_checks(topk_ids, expert_to_rank, T, K, E, workspace);
  if (st != HM_OK) return st;
  if (!hm::swap_cuts_ok(G, ncuts, ng)) return HM_ERR_TOPOLOGY;
  for (int c = 0; c < ncuts; ++c)
    if (!Z[c]) return HM_ERR_NULL;
  if (workspace_bytes < hm_swap_multi_workspace_bytes(T, K, E, G, ncuts, ng)) return HM_ERR_WORKSPACE;
  return hm::swap_counts_launch(topk_ids, expert_to_rank, T, K, E, G, ncuts, ng, Z, status, workspace, (hipStream_t)hip_stream);
}

extern "C" size_t hm_swap_select_workspace_bytes(int32_t E) {
  if (E < 1) return 0;
  const int64_t blocks = ((int64_t)E * E + hm::kSelectPairs - 1) / hm::kSelectPairs;
  return (size_t)blocks * (sizeof(double) + sizeof(int32_t)) + 16;
}

extern "C" hm_status hm_swap_select(int32_t d, const int32_t *U, int32_t G, int32_t E, double M, double v,
                                    const int32_t *const *z_inter, const int32_t *z_intra, const double *scale_inter,
                                    double scale_intra, const double *alpha_inter, const double *beta_inter,
                                    double alpha_intra, double beta_intra, double gamma, double *Q, int32_t *best_pair,
                                    double *best_time, void *workspace, size_t workspace_bytes, void *hip_stream) {
  HM_ENTRY_SCOPE;
  using namespace hm;
  if (!U || !z_intra || !Q || !best_pair || !best_time || !workspace) return HM_ERR_NULL;
  if (d < 1 || d > kMaxDim || G < 1 || G > 64 || U[0] != 1) return HM_ERR_TOPOLOGY;
  if (E < 1 || (int64_t)E * E > 2147483647LL) return HM_ERR_SHAPE;
  if (d > 1 && (!z_inter || !scale_inter || !alpha_inter || !beta_inter)) return HM_ERR_NULL;
  for (int i = 1; i < d; ++i) {
    if (!z_inter[i]) return HM_ERR_NULL;
    if (U[i] < U[i - 1] || U[i] > G || U[i] % U[i - 1] != 0 || G % U[i] != 0) return HM_ERR_TOPOLOGY;
  }
  if (workspace_bytes < hm_swap_select_workspace_bytes(E)) return HM_ERR_WORKSPACE;
  SelectParams p;
  p.d = d;
  p.G = G;
  p.E = E;
  p.M = M;
  p.v = v;
  p.gamma = gamma;
  for (int i = 0; i < kMaxDim; ++i) {
    const bool in = i >= 1 && i < d;
    p.U[i] = i < d ? U[i] : 1;
    p.z_inter[i] = in ? z_inter[i] : nullptr;
    p.scale_inter[i] = in ? scale_inter[i] : 0.0;
    p.alpha_inter[i] = in ? alpha_inter[i] : 0.0;
    p.beta_inter[i] = in ? beta_inter[i] : 0.0;
  }
  p.z_intra = z_intra;
  p.scale_intra = scale_intra;
  p.alpha_intra = alpha_intra;
  p.beta_intra = beta_intra;
  p.Q = Q;
  p.nblocks = (int32_t)(((int64_t)E * E + kSelectPairs - 1) / kSelectPairs);
  p.block_min = (double *)workspace;
  p.block_arg = (int32_t *)(p.block_min + p.nblocks);
  p.best_pair = best_pair;
  p.best_time = best_time;
  hipStream_t stream = (hipStream_t)hip_stream;
  hipLaunchKernelGGL(G <= 32 ? swap_q_kernel<32> : swap_q_kernel<64>, dim3(p.nblocks), dim3(kSelectThreads), 0, stream, p);
  if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  hipLaunchKernelGGL(swap_argmin_kernel, dim3(1), dim3(kArgminThreads), 0, stream, p);
  return hm_launch_status();
}

extern "C" hm_status hm_swap_apply(int32_t *expert_to_rank, int32_t E, const int32_t *best_pair, void *hip_stream) {
  HM_ENTRY_SCOPE;
  if (!expert_to_rank || !best_pair) return HM_ERR_NULL;
  if (E < 1) return HM_ERR_SHAPE;
  hipLaunchKernelGGL(hm::swap_apply_kernel, dim3(1), dim3(hm::kWave), 0, (hipStream_t)hip_stream, expert_to_rank, E,
                     best_pair);
  return hm_launch_status();
}
