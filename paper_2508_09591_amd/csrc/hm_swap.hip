// Hierarchical expert swap (HierMoE Section IV): the swap tensor Z and the selection of Eq.(8)-(11).
//
// Z[r][c][:] is the vector of duplicate-free per-group token counts after experts r and c trade
// places.  A swap can only change the two groups involved, and by how much follows from three
// small co-occurrence tables over the tokens:
//   L0[a]    tokens selecting a                      CG[a][g]  ... that also select something in g
//   L[a]     tokens where a is alone in its group    C[a][b]   ... that also select b
// For g_r != g_c:  Z[r][c][g_c] = base[g_c] + (L0[r] - CG[r][g_c]) - (L[c] - C[c][r])   and the same
// with r and c exchanged for g_r: no O(T K E) walk over all unselected experts, and the per-pair
// work is an embarrassingly parallel E^2 ng kernel.  The tables come from matrix products on
// the matrix cores for E <= 512 (further down), from O(T K (K + ng)) atomic updates, one lane per
// routing slot, beyond that, for E > 256 with more than eight slots per token, and where the products would have
// too little to do (atomics_pay).
#include "hm_cooc.h"
#include "hm_device.h"

#include <type_traits>

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
  int32_t build_blocks[kMaxCuts];     // column blocks of swap_build_kernel per cut
  int32_t lds_off[kMaxCuts];   // ints: where cut c's [L (E) | CG (E * ng)] starts in LDS; L0 is at 0
  int32_t *L0;                 // [E]                                  (workspace, shared by the cuts)
  int32_t *base[kMaxCuts];     // [64]                                 (workspace, per cut)
  int32_t *L[kMaxCuts];        // [E]
  int32_t *CG[kMaxCuts];       // [E][ng]
  int32_t *C[kMaxCuts];        // [copies][E][E]
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
// expert of its group, and M[t][g] = 1 when t selects something in group g (all 0 or 1):
//   C  = A^T S   (its diagonal is L)        CG = S^T M   (L0[a] = CG[a][group of a])
// so the read-modify-write updates of popular expert pairs, which serialise on one address, become
// matrix products whose sums are held in registers.  A workgroup takes one cut, a contiguous chunk of the tokens and
// a panel of columns of C, builds the three indicator tiles in LDS (expert-major, a mark is a nibble: 1.0 in FP4, so that
// a lane's MFMA operand of 32 tokens is 16 contiguous bytes and 1,024 tokens of 128 experts fit at once), and stores
// its partial tables with plain stores; swap_pairs_kernel sums the chunks where it puts Z together.  The products add up
// zeros and ones in binary32, which is exact below 2^24; a chunk has fewer than 2^15 tokens, or, added, at most 2^24.
// (With many tokens, or E > 256, for which the workspace has no room for partial tables, the chunks are added to
// cleared tables by atomics, or the slots are: atomics_pay.)
// ---------------------------------------------------------------------------------------------
// Partial tables per cut, some of them of no token where there are few: whoever sums them need not ask how many there are.
constexpr int kCoocChunks = 16;
constexpr int kCoocChunkTokensMax = 32640;   // a chunk's counts are stored as 16-bit values
constexpr int kCoocAddedTokensMax = 1 << 24; // a workgroup's sums are binary32
constexpr int kCoocMaxE = 512;
// Workgroups aimed at where chunks are added up, one per CU: fewer leave CUs idle, more add more tables (E = 320, four
// cuts, K = 8, with 128 / 256 / 512: 4,096 tokens 22.0 / 21.7 / 28.0 us, 16,384 40.0 / 31.5 / 38.2, 300,000 443 / 231 /
// 226).
constexpr int kCoocAddedGroups = 256;
constexpr int kCoocOwnK = 8;         // most slots of a token that the matrix kernel works out itself
constexpr int kCoocThreads = kCoocWaves * kWave;   // = most tokens of a tile: a lane per token
constexpr int kCoocStep = 64;        // tokens of one 32x32x64 product
constexpr int kCoocPad = 16;         // bytes behind a tile row, which spread 32 rows over all banks
constexpr int kCoocLds = 162816;     // dynamic LDS of a workgroup, most
constexpr int kBlock = 16;           // experts of a block of the tables

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef i32x4 i32x4_align4 __attribute__((aligned(4)));
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef u16x4 u16x4_align2 __attribute__((aligned(2)));

struct CoocParams {
  const int32_t *ids;
  const int32_t *expert_to_rank;
  int32_t T, K, E, G;
  int32_t sub_log2;            // lanes per token of swap_slots_kernel: 2^sub_log2 >= K
  int32_t ncuts;
  int32_t chunks;              // gridDim.x of the matrix kernel
  int32_t tokens_per_chunk;    // a multiple of kCoocStep
  int32_t tile_tokens, stride; // tokens of a tile, bytes of a tile row
  uint32_t per_recip16[kMaxCuts];   // ceil(2^16 / per): exact for ranks (below 64)
  uint32_t words_recip17;      // ceil(2^17 / (tile_tokens / 8))
  uint32_t k_reciprocal;       // ceil(2^32 / K) for K > 1
  int32_t ng[kMaxCuts], per[kMaxCuts];
  uint8_t *slot_bits;          // [T * K]: bit 0 first valid occurrence, bit 1 + c alone in its group under cut c
  void *tables[kMaxCuts];      // 16-bit counts of every chunk (parts) or 32-bit counts, as Tables lays them out
  int32_t *status;
};

// The tables of a cut, in blocks of up to 16 experts a (h of them) by up to 16 columns, chunk by chunk, a block's
// values with the experts side by side: [C: E blocks by E][CG: E by ng][L: E][base: 64].  A block of all chunks is
// contiguous, so whoever sums the chunks of a block reads whole lines, and four neighbouring experts of a lane's
// accumulators are one store. Tables that chunks are added to are plain rows, [C: E by E][CG: E by ng][L][base], as the
// lanes of an atomic should be neighbours.
struct Tables {
  int E, ng, chunks;
  __host__ __device__ static int64_t values(int64_t E, int64_t ng) { return E * E + E * ng + E + 64; }   // of a chunk
  __device__ int height(int i) const { return min(kBlock, E - kBlock * i); }
  // Where block i of a table begins, and a column or chunk of columns from there, in heights of the block.
  __device__ int c(int i) const { return kBlock * i * E * chunks; }
  __device__ int c_column(int b, int chunk) const { return b / kBlock * kBlock * chunks + chunk * height(b / kBlock) + b % kBlock; }
  __device__ int cg(int i) const { return (E * E + kBlock * i * ng) * chunks; }
  __device__ int cg_column(int g, int chunk) const { return chunk * ng + g; }
  __device__ int l(int i) const { return (E * E + E * ng + kBlock * i) * chunks; }   // columns: chunks
  __device__ int base(int chunk) const { return (E * E + E * ng + E) * chunks + chunk * kWave; }
};

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

// D += A B for one 32x32 tile over 64 tokens; a lane's operand: 32 tokens, FP4, of row (lane % 32).
__device__ __forceinline__ f32x16 mfma_fp4(i32x4 a, i32x4 b, f32x16 acc) {
  const i32x8 a8 = {a[0], a[1], a[2], a[3], 0, 0, 0, 0}, b8 = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, acc, 4, 4, 0, 0, 0, 0);   // 4: FP4; no scales
}
constexpr uint32_t kOne = 2;   // 1.0 in FP4

// An expert's group as the matrix kernel looks it up: below 64, or one of these.
constexpr uint32_t kNoGroup = 0x80, kBadGroup = 0xC0;   // id -1; an id or a placement out of range

// A product below 2^24: one instruction at the full rate.
__device__ __forceinline__ int row_at(uint32_t row, int stride) { return (int)__umul24(row, (uint32_t)stride); }

// The marks of a lane's token of up to eight slots, written for few instructions: the sixteen waves of a workgroup
// issue each of them in turn.  Groups are bits of BITS: one that has been seen twice, copies of an expert aside, is
// nobody's alone.  `m`, `a`: the token's word in row 0 of the tiles, a_to_s: from an expert's row of A to its row of S,
// `value`: the token's bit.
template <typename BITS>
__device__ __forceinline__ void mark_token(const int (&id)[kCoocOwnK], int E, const uint8_t *group_of, int stride, int panel0,
                                           int panel, uint8_t *m, uint8_t *a, int a_to_s, uint32_t value, bool &bad) {
  uint32_t expert[kCoocOwnK], group[kCoocOwnK], all = 0;
  uint32_t same = 1;   // 0 if two slots have one expert
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k)   // entry 0: id -1, E + 1: out of range
    group[k] = group_of[min((uint32_t)id[k] + 1u, (uint32_t)E + 1u)];
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) {
    all |= group[k];
    expert[k] = group[k] < kWave ? (uint32_t)id[k] : 0x10000u + k;   // equal to no other
#pragma unroll
    for (int j = 0; j < k; ++j) same = min(same, expert[j] ^ expert[k]);
  }
  bad = bad || (all & kBadGroup & ~kNoGroup) != 0;
  BITS bit[kCoocOwnK], once = 0, twice = 0;
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) bit[k] = group[k] < kWave ? (BITS)1 << (group[k] & (8 * sizeof(BITS) - 1)) : (BITS)0;
  if (__builtin_expect(__ballot(same == 0) != 0, 0)) {   // routers do not select an expert twice, callers may
#pragma unroll
    for (int k = 1; k < kCoocOwnK; ++k) {
      bool again = false;
#pragma unroll
      for (int j = 0; j < k; ++j) again = again || expert[j] == expert[k];
      if (again) bit[k] = 0;
    }
  }
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) {
    twice |= once & bit[k];
    once |= bit[k];
  }
#pragma unroll
  for (int k = 0; k < kCoocOwnK; ++k) {
    const bool marks = bit[k] != 0;   // another copy of an expert has the same marks
    const uint32_t column = expert[k] - (uint32_t)panel0;
    atomicOr((uint32_t *)(m + row_at(group[k] & (kWave / 2 * sizeof(BITS) / 4 - 1), stride)), marks ? value : 0u);
    uint8_t *const row = a + row_at(expert[k], stride);
    if (marks && column < (uint32_t)panel) atomicOr((uint32_t *)(row + a_to_s), value);
    if ((bit[k] & ~twice) != 0) atomicOr((uint32_t *)row, value);
  }
}

// Four neighbouring values of a block, as far as they are below `left`.
__device__ __forceinline__ void store_four(uint16_t *out, const int (&v)[4], int left) {
  if (left >= 4) {
    *(u16x4_align2 *)out = (u16x4){(uint16_t)v[0], (uint16_t)v[1], (uint16_t)v[2], (uint16_t)v[3]};
  } else {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (i < left) out[i] = (uint16_t)v[i];
  }
}
// Workgroup (chunk, cut, panel of 32 COLS columns of C); a wave holds one row of 32x32 tiles of the panel, the last
// waves a tile of its CG each.  A workgroup needs the S tile of its own columns only; the panels repeat the marks of
// the chunk's slots and the A tile.  One column of tiles up to 128 experts, so that four cuts and sixteen chunks are a
// workgroup per CU, two for 256, one again beyond, where a wave per tile row is all there are.
//
// Per tile of up to 1,024 tokens: load and clear | barrier | mark | barrier | multiply, and a barrier if there are more
// tiles.  All marks of a chunk of that many tokens are made at once: with a byte per mark a tile held 128, and the
// chain of marks, barrier, LDS operands, products and barrier, 0.5 us per tile, was half of the kernel.  What bounds it
// now is the marks, which sixteen waves issue in turn, 1.0 to 1.7 us of 7 (products 0.6, clearing 0.5, stores 0.6), and
// cold code, 8 KB of it.  Kernel trace, four cuts, K = 8, bytes -> nibbles: 16,384 tokens, 128 experts 11.8 -> 6.6 us,
// 8,192, 256 12.2 -> 7.9.  The whole call (graphs of ten), 4,096, 65,536, 500,000 tokens: 128 experts 16.0 -> 11.4,
// 42.4 -> 21.3, 223 -> 97; 256 25.8 -> 18.5, 57.7 -> 35.6, 272 -> 151.
template <int COLS, bool OWN_SLOTS, bool ADDED>   // ADDED: to cleared tables, instead of stored as a part
__global__ __launch_bounds__(kCoocThreads) void swap_cooc_kernel(CoocParams p) {
  constexpr int kPanel = 32 * COLS, kAhead = 4 / COLS;   // products whose operands are on their way together
  constexpr bool kBoth = ADDED && COLS == 1;             // more than 448 experts: the last waves have tiles of C and of CG
  typedef std::conditional_t<ADDED, int32_t, uint16_t> value_t;
  extern __shared__ __align__(16) uint8_t tiles[];
  __shared__ uint8_t group_of[kCoocMaxE + 2];   // of expert e at e + 1
  __shared__ int32_t base_cnt[kWave];

  const int cut = blockIdx.y, panel = blockIdx.z, chunk = blockIdx.x;
  const int E = p.E, ng = p.ng[cut], stride = p.stride;
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  typedef CoocTiles<COLS> layout_t;
  const layout_t lay(E, ng);
  // rows of `stride` bytes
  uint8_t *const a_tile = tiles, *const s_tile = tiles + lay.s_at() * stride, *const m_tile = tiles + lay.m_at() * stride;
  const int vecs = lay.rows() * (stride / 16);

  // Where a token of the tile is marked: in the row's word (token % words) and there in nibble (token / words), so that
  // the lanes of a wave, which hold neighbouring tokens, meet at a bank only where their rows do, and never at a word.
  // The products take the tokens in any order.
  const int words = p.tile_tokens >> 3;
  auto place = [&](int token, int &at) {
    const uint32_t nibble = __umul24((uint32_t)token, p.words_recip17) >> 17;   // token < 1,024, 16 to 128 words
    at = (token - (int)__umul24(nibble, (uint32_t)words)) * 4;
    return kOne << (4 * nibble);
  };

  // What this wave accumulates: a row of tiles of C, or, from the last wave down, one tile of the panel's CG.
  const bool has_c = lay.has_c(w), has_g = lay.has_g(w);
  const int quarter = w - kCoocWaves / 2;   // of the tokens whose groups the wave counts, a lane per group
  const bool counts_base = panel == 0 && (unsigned)quarter < 4u;
  f32x16 acc[COLS], second;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (kBoth) second[r] = 0.0f;
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[c][r] = 0.0f;
  }
  int my_base = 0;
  if (tid < kWave) base_cnt[tid] = 0;
  const int op_at = (lane & 31) * stride + (lane >> 5) * 16, steps = p.tile_tokens / kCoocStep;   // whole batches
  // acc[c] += rows' tile by the tile of columns c
  auto multiply = [&](auto &sums, const uint8_t *rows, const uint8_t *columns) {
    constexpr int N = sizeof(sums) / sizeof(f32x16);
    rows += op_at;
    columns += op_at;
#pragma unroll 1
    for (int step = 0; step < steps; step += kAhead, rows += 32 * kAhead, columns += 32 * kAhead) {
      i32x4 r_op[kAhead], c_op[kAhead][N];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        r_op[j] = *(const i32x4 *)(rows + 32 * j);
#pragma unroll
        for (int c = 0; c < N; ++c) c_op[j][c] = *(const i32x4 *)(columns + 32 * c * stride + 32 * j);
      }
#pragma unroll
      for (int j = 0; j < kAhead; ++j)
#pragma unroll
        for (int c = 0; c < N; ++c) sums[c] = mfma_fp4(r_op[j], c_op[j][c], sums[c]);
    }
  };
  // the tile rows and columns of this wave's products
  const uint8_t *const rows = tiles + (has_c ? lay.c_rows(w) : lay.g_rows(w)) * stride;
  const uint8_t *const columns = tiles + (has_c ? lay.c_columns(w) : lay.g_columns(w)) * stride;

  const uint32_t T = (uint32_t)p.T, t_begin = (uint32_t)chunk * (uint32_t)p.tokens_per_chunk;
  const uint32_t t_end = min(T, t_begin + (uint32_t)p.tokens_per_chunk);
  bool bad = false;
#pragma unroll 1
  for (uint32_t t0 = t_begin; t0 < t_end; t0 += (uint32_t)p.tile_tokens) {
    const int tokens = (int)min((uint32_t)p.tile_tokens, t_end - t0);
    int id[kCoocOwnK], rank = -1;
    if (OWN_SLOTS) {   // on their way, as the placement, while the tiles are cleared
#pragma unroll
      for (int k = 0; k < kCoocOwnK; ++k) id[k] = -1;
      if (tid < tokens) load_ids(p.ids + (int64_t)(t0 + (uint32_t)tid) * p.K, p.K, 0, id);
    }
    if (t0 == t_begin && tid >= 1 && tid <= E) rank = p.expert_to_rank[tid - 1];
    if (t0 != t_begin) __syncthreads();
    const i32x4 zero = {0, 0, 0, 0};
#pragma unroll 1
    for (int i = tid; i < vecs; i += kCoocThreads) ((i32x4 *)tiles)[i] = zero;
    if (t0 == t_begin) {
      if (tid < E + 2)
        group_of[tid] = (uint8_t)(tid == 0                            ? kNoGroup
                                  : (unsigned)rank < (unsigned)p.G ? __umul24((uint32_t)rank, p.per_recip16[cut]) >> 16
                                                                   : kBadGroup);
    }
    __syncthreads();
    if (OWN_SLOTS) {
      if (w * kWave < tokens) {
        int at;
        const uint32_t value = place(tid, at);
        const int a_to_s = (lay.s_at() - kPanel * panel) * stride;
        const int panel0 = kPanel * panel;
        if (__builtin_expect(ng <= 32, 1))
          mark_token<uint32_t>(id, E, group_of, stride, panel0, kPanel, m_tile + at, a_tile + at, a_to_s, value, bad);
        else
          mark_token<uint64_t>(id, E, group_of, stride, panel0, kPanel, m_tile + at, a_tile + at, a_to_s, value, bad);
      }
    } else {
      constexpr int kLoads = 8;   // of a lane in flight together
      const int slots = tokens * p.K;
      const int32_t *const ids = p.ids + (int64_t)t0 * p.K;
      const uint8_t *const slot_bits = p.slot_bits + (int64_t)t0 * p.K;
#pragma unroll 1
      for (int i0 = tid; i0 < slots; i0 += kLoads * kCoocThreads) {
        int expert[kLoads], bits[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
          const int i = min(i0 + j * kCoocThreads, slots - 1);
          expert[j] = ids[i];
          bits[j] = slot_bits[i];
        }
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
          const int i = i0 + j * kCoocThreads;
          if (i < slots && (bits[j] & 1)) {   // a valid expert
            int at;
            const uint32_t value = place((int)__umulhi((uint32_t)i, p.k_reciprocal), at);
            const uint32_t column = (uint32_t)(expert[j] - kPanel * panel);
            atomicOr((uint32_t *)(m_tile + row_at(group_of[expert[j] + 1], stride) + at), value);
            if (column < (uint32_t)kPanel) atomicOr((uint32_t *)(s_tile + row_at(column, stride) + at), value);
            if ((bits[j] >> (1 + cut)) & 1) atomicOr((uint32_t *)(a_tile + row_at((uint32_t)expert[j], stride) + at), value);
          }
        }
      }
    }
    __syncthreads();
    auto of_g = [](f32x16 &sums) -> f32x16(&)[layout_t::kColumnsOfG] { return *(f32x16(*)[layout_t::kColumnsOfG])&sums; };
    if (layout_t::kColumnsOfC == layout_t::kColumnsOfG) {
      if (has_c || has_g) multiply(acc, rows, columns);
    } else {
      // One tile of CG, not COLS: behind M's tiles LDS ends (200,000 tokens, 256 experts, four cuts: with a second product,
      // of the same tile, whose sums are dropped, 76.6 us, 71.8 without; 8,192 18.9 and 18.7).
      if (has_c) multiply(acc, rows, columns);
      else if (has_g) multiply(of_g(acc[0]), rows, columns);
    }
    if (kBoth && has_c && has_g) multiply(of_g(second), tiles + lay.g_rows(w) * stride, tiles + lay.g_columns(w) * stride);
    if (counts_base) {   // a mark is one bit, so a word's population count is its number of tokens
      const i32x4 *row = (const i32x4 *)(m_tile + min(lane, 32 * lay.m - 1) * stride);
#pragma unroll 1
      for (int i = quarter; i < 2 * steps; i += 4) {
        const i32x4 v = row[i];
        my_base += __popc(v[0]) + __popc(v[1]) + __popc(v[2]) + __popc(v[3]);
      }
    }
  }
  if (OWN_SLOTS && bad && cut == 0 && panel == 0) flag(p.status, HM_ERR_BAD_ID);

  // Accumulator layout of a 32x32 tile: register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4,
  // column l % 32.
  const Tables table = {E, ng, ADDED ? 1 : p.chunks};
  const int part = ADDED ? 0 : chunk, col = lane & 31, row_hi = (lane >> 5) * 4;
  value_t *const out = (value_t *)p.tables[cut];
  // the four 4 x 1 pieces of a lane's column of the tile whose first block is `block`: where the table begins, its width, the
  // column, for parts in heights
  auto put = [&](const f32x16 &sums, int block, int begin, int width, int column) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int h = table.height(block + q / 2), row = 8 * (q & 1) + row_hi;
      if (row >= h) continue;
      const int v[4] = {(int)sums[4 * q], (int)sums[4 * q + 1], (int)sums[4 * q + 2], (int)sums[4 * q + 3]};
      if constexpr (ADDED) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < h - row && v[i]) atomicAdd(out + begin + (kBlock * (block + q / 2) + row + i) * width + column, v[i]);
      } else {
        value_t *const at = out + (begin + (block + q / 2) * kBlock * width * table.chunks);
        store_four(at + ((int)__umul24((uint32_t)h, (uint32_t)column) + row), v, h - row);
      }
    }
  };
  auto put_groups = [&](const f32x16 &sums) {
    const int g = 32 * lay.g_column(w) + col;
    if (g < ng) put(sums, (kPanel * panel + 32 * lay.g_row(w)) / kBlock, table.cg(0), ng, ADDED ? g : table.cg_column(g, part));
  };
  if (has_c) {
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      const int b = kPanel * panel + 32 * c + col;
      if (b >= E) continue;
      put(acc[c], 2 * w, 0, E, ADDED ? b : table.c_column(b, part));
      if (kPanel * panel + 32 * c == 32 * w && (col & 4) == row_hi) {   // the diagonal: row = col
        float diagonal = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) diagonal = (col >> 3) * 4 + (col & 3) == r ? acc[c][r] : diagonal;
        value_t *const at = out + table.l(b / kBlock) + part * table.height(b / kBlock) + b % kBlock;
        if constexpr (!ADDED) *at = (uint16_t)(int)diagonal;
        else if (diagonal != 0.0f) atomicAdd(at, (int)diagonal);
      }
    }
    if (kBoth && has_g) put_groups(second);
  } else if (has_g) {
    put_groups(acc[0]);
  }
  if (panel != 0) return;
  __syncthreads();   // a chunk without a token has had none
  if (counts_base && lane < ng && my_base) atomicAdd(&base_cnt[lane], my_base);
  __syncthreads();
  if (tid < kWave) {
    if constexpr (!ADDED) out[table.base(part) + tid] = (uint16_t)base_cnt[tid];
    else if (base_cnt[tid]) atomicAdd(out + table.base(part) + tid, base_cnt[tid]);
  }
}

// Z from the tables: a workgroup takes the pairs of two blocks of up to 16 experts, (r, c) and (c, r), as Z[r][c] =
// Z[c][r]. It sums the chunks of what these pairs need (two blocks of C, the CG rows of 32 experts, every value of C
// once for the whole chip), puts the two changed counts of every pair together in LDS, and writes both orientations.
// What bounds it is waiting: by the counters its waves wait for memory, LDS or one another 59 % of their time with 128
// experts and 48 % with 256, for an instruction to be fetched or issued 16 % and 32 %; their vector instructions (some
// 250 a wave) take 0.5 us and 2.0 us of the SIMDs' time, and it writes Z and nothing else.  Kernel trace, 128 experts,
// 16,384 tokens, four cuts: a kernel that summed the chunks and wrote transposes of C and CG, and one that looked them
// up per value of Z, 4.4 + 5.7 us, now 6.2; 256 experts, 8,192 tokens (15.7 MB of Z) 6.2 + 7.6, now 9.0.
constexpr int kPairThreads = 512;
struct PairCut {
  const void *tables;
  int32_t *Z;
  int32_t ng;
  uint32_t per_recip16;   // ceil(2^16 / ranks of a group): exact for ranks (below 64)
  int32_t wide, of_pair;                  // groups of a lane's store, 4 or 1; lanes that take a pair: ng / wide
  int32_t of_pair_recip20, pairs_at_once;   // ceil(2^20 / of_pair), kPairThreads / of_pair
};
struct PairParams {
  const int32_t *expert_to_rank;
  int32_t *status;
  int32_t E, G, ncuts, blocks;   // blocks of experts
  PairCut cut[kMaxCuts];
};
__device__ __forceinline__ i32x4 load_four(const int32_t *at) { return *(const i32x4_align4 *)at; }
__device__ __forceinline__ u16x4 load_four(const uint16_t *at) { return *(const u16x4_align2 *)at; }

// N chunks, every STEP-th, of four values that begin at i of the n of a chunk; `at` is the first of these chunks.  The
// sums are of 32 bits; counts of 16 come two in a word, and a product with (1, 0) or (0, 1) adds one of them in an
// instruction (the whole call, 128 experts, four cuts, 8,192 tokens 11.9 us, with a conversion of each count 12.2, with
// sums of 16 bits, two in an instruction, 11.9; 256 experts 19.1, 19.4, 18.8).
template <int N, int STEP, typename V>
struct Chunks {
  decltype(load_four((const V *)nullptr)) v[N];
  __device__ __forceinline__ void load(const V *at, int n, int i) {
    const uint32_t bytes = (uint32_t)i * sizeof(V);
#pragma unroll
    for (int j = 0; j < N; ++j, at += STEP * n) v[j] = load_four((const V *)((const char *)at + bytes));
  }
  __device__ __forceinline__ void sum(int32_t *out) const {
    i32x4 s = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if constexpr (sizeof(V) == sizeof(uint16_t)) {
        typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const u16x2 word = {v[j][e & 2], v[j][e | 1]}, half = {(uint16_t)(~e & 1), (uint16_t)(e & 1)};
          s[e] = (int32_t)__builtin_amdgcn_udot2(word, half, (uint32_t)s[e], false);
        }
      } else {
        s += v[j];
      }
    }
    *(i32x4_align4 *)out = s;
  }
};
// Blocks of fewer than four values (the last of a few experts with a few groups): a lane per value.
template <typename V>
__device__ __forceinline__ void sum_few(int32_t *out, const V *at, int n, int i, int count, int step) {
  if (i >= n) return;
  int sum = 0;
  for (int c = 0; c < count; ++c) sum += at[c * step * n + i];
  out[i] = sum;
}

// V: type of a count in the tables.
template <typename V, int CHUNKS>   // one chunk: tables that chunks were added to
__global__ __launch_bounds__(kPairThreads) void swap_pairs_kernel(PairParams p) {
  constexpr int kOfC = CHUNKS > 4 ? 4 : 1, kOfCG = CHUNKS > 4 ? 2 : 1;   // waves that share the chunks of a value
  __shared__ __align__(16) int32_t s_c[2][kOfC][kBlock * kBlock];    // [block (I, J), (J, I)]
  __shared__ __align__(16) int32_t s_cg[2][kOfCG][kBlock * kWave];   // [block I, J][group][expert]
  __shared__ __align__(16) i32x4 s_pair[kBlock][kBlock + 1];         // [r][c]: what the groups of c and of r gain, and which they are
  __shared__ int32_t s_l[2 * kBlock], s_group[2 * kBlock], s_base[kWave];   // of I, of J

  const PairCut cut = p.cut[p.ncuts - 1 - (int)blockIdx.z];   // the last cut first: usually the finest, whose workgroups last longest
  const int ng = cut.ng, E = p.E, blocks = p.blocks;
  // every unordered pair of blocks once: (I, I + y) round the circle, of the opposite ones half
  const int I = blockIdx.x, y = blockIdx.y, J = I + y < blocks ? I + y : I + y - blocks;
  if (2 * y == blocks && I >= y) return;
  const Tables table = {E, ng, CHUNKS};
  const V *const part = (const V *)cut.tables;
  const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int height_i = table.height(I), height_j = table.height(J);

  // Waves 0 to 3 have block (I, J) of C and the CG of I, 4 to 7 block (J, I) and J.  Every load is on its way before
  // the first is used.
  const int side = w >> 2, of_c = w & (kOfC - 1), of_cg = w >> 1 & (kOfCG - 1);
  const int n_c = height_i * height_j, n_cg = (side ? height_j : height_i) * ng;
  // the last four may be values of another lane, too
  const int c_i = min(4 * lane, n_c - 4), q0 = (w & 1) * kWave + lane, cg_i = min(4 * q0, n_cg - 4);
  const int rows_of = side ? J : I, cols_of = side ? I : J, rows = side ? height_j : height_i, cols = side ? height_i : height_j;
  const V *const c_at = part + table.c(rows_of) + rows * table.c_column(kBlock * cols_of, of_c);
  const V *const cg_at = part + table.cg(rows_of) + rows * table.cg_column(0, of_cg);
  Chunks<CHUNKS / kOfC, kOfC, V> c;
  Chunks<CHUNKS / kOfCG, kOfCG, V> cg;
  V plain = 0;   // of plain rows: a value of the block per lane of its waves
  if (CHUNKS > 1) {
    if (n_c >= 4) c.load(c_at, n_c, c_i);
  } else {
    const int i = tid & (kBlock * kBlock - 1);
    plain = part[(kBlock * rows_of + min(i & (kBlock - 1), rows - 1)) * E + kBlock * cols_of + min(i >> 4, cols - 1)];
  }
  if (n_cg >= 4) cg.load(cg_at, n_cg, cg_i);
  const int a = lane & (kBlock - 1), of_j = lane >> 4 & 1, h = of_j ? height_j : height_i;
  int l = 0, base[2] = {0, 0}, rank = -1;   // of one chunk or two
  {
    const int chunk = 2 * w + (lane >> 5);
    if (chunk < CHUNKS && a < h) l = part[table.l(of_j ? J : I) + chunk * h + a];
    if (w < CHUNKS) base[0] = part[table.base(w) + lane];
    if (CHUNKS > kPairThreads / kWave) base[1] = part[table.base(w + kPairThreads / kWave) + lane];
    if (w == 0 && lane < 2 * kBlock && a < h) rank = p.expert_to_rank[kBlock * (of_j ? J : I) + a];
  }
  __builtin_amdgcn_sched_barrier(0);
  if (CHUNKS == 1) {
    const int i = tid & (kBlock * kBlock - 1), row = i & (kBlock - 1), col = i >> 4;
    if (row < rows && col < cols) s_c[side][0][col * rows + row] = (int)plain;
  } else if (n_c >= 4) c.sum(&s_c[side][of_c][c_i]);
  else sum_few(s_c[side][of_c], c_at, n_c, lane, CHUNKS / kOfC, kOfC);
  if (__builtin_expect(n_cg < 4, 0)) {
    sum_few(s_cg[side][of_cg], cg_at, n_cg, q0, CHUNKS / kOfCG, kOfCG);
  } else {
    cg.sum(&s_cg[side][of_cg][cg_i]);
    if (__builtin_expect(n_cg > 8 * kWave, 0)) {   // more than 32 groups
      const int i = min(4 * (q0 + 2 * kWave), n_cg - 4);
      cg.load(cg_at, n_cg, i);
      cg.sum(&s_cg[side][of_cg][i]);
    }
  }
  if (tid < 2 * kBlock) s_l[tid] = 0;
  if (tid < kWave) s_base[tid] = 0;
  __syncthreads();
  if (l) atomicAdd(&s_l[lane & (2 * kBlock - 1)], l);
  if (base[0] + base[1]) atomicAdd(&s_base[lane], base[0] + base[1]);
  if (tid < 2 * kBlock) {
    s_group[tid] = (unsigned)rank < (unsigned)p.G ? (int)(((uint32_t)rank * cut.per_recip16) >> 16) : -1;
  }
  __syncthreads();

  if (tid < kBlock * kBlock) {
    const int r = tid & (kBlock - 1), c = tid >> 4;
    if (r < height_i && c < height_j) {
      const int gr = s_group[r], gc = s_group[kBlock + c];
      i32x4 pair = {0, 0, -1, -1};
      if (gr < 0 || gc < 0) flag(p.status, HM_ERR_BAD_ID);
      if (gr >= 0 && gc >= 0 && gr != gc) {
        int gain_c = -s_l[kBlock + c], gain_r = -s_l[r];
#pragma unroll
        for (int i = 0; i < kOfC; ++i) {
          gain_c += s_c[1][i][r * height_j + c];   // C[c][r]
          gain_r += s_c[0][i][c * height_i + r];   // C[r][c]
        }
#pragma unroll
        for (int i = 0; i < kOfCG; ++i) {
          auto of_r = [&](int g) { return s_cg[0][i][CHUNKS > 1 ? g * height_i + r : r * ng + g]; };
          auto of_c = [&](int g) { return s_cg[1][i][CHUNKS > 1 ? g * height_j + c : c * ng + g]; };
          gain_c += of_r(gr) - of_r(gc);   // L0[r] - CG[r][gc]
          gain_r += of_c(gc) - of_c(gr);
        }
        pair = (i32x4){gain_c, gain_r, gc, gr};
      }
      s_pair[r][c] = pair;
    }
  }
  __syncthreads();

  // `of_pair` neighbouring lanes take a pair, a lane the same groups of every pair it takes.
  const int of_pair = cut.of_pair, wide = cut.wide;
  const int first = (int)((uint32_t)tid * (uint32_t)cut.of_pair_recip20 >> 20), j = wide * (tid - first * of_pair);
  const int at_once = cut.pairs_at_once;
  if (first >= at_once) return;
  i32x4 base4;
#pragma unroll
  for (int e = 0; e < 4; ++e) base4[e] = s_base[min(j + e, kWave - 1)];
#pragma unroll 1
  for (int turned = 0; turned < (I == J ? 1 : 2); ++turned) {
    const int cols = turned ? height_i : height_j, pairs = height_i * height_j;
    const uint32_t recip16 = cols == kBlock ? 65536u / kBlock : (65536u + (uint32_t)cols - 1u) / (uint32_t)cols;
    int32_t *const out = cut.Z + ((int64_t)(kBlock * (turned ? J : I)) * E + kBlock * (turned ? I : J)) * ng + j;
#pragma unroll 1
    for (int i = first; i < pairs; i += at_once) {
      const int row = (int)((uint32_t)i * recip16 >> 16), col = i - row * cols;
      const i32x4 pair = turned ? s_pair[col][row] : s_pair[row][col];
      i32x4 z = base4;
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] += (pair[2] == j + e ? pair[0] : 0) + (pair[3] == j + e ? pair[1] : 0);
      int32_t *const at = out + (row * E + col) * ng;
      if (wide == 4) *(i32x4_align4 *)at = z;
      else *at = z[0];
    }
  }
}

// Z by the atomics' tables: one lane per (c, j) of a cut and kBuildRows row experts r: blockIdx.y is the block of rows and
// blockIdx.x runs over the column blocks (256 consecutive (c, j)) of all cuts, one cut after the
// other.  The loads of all rows are issued before the first value is put together, so a lane
// waits for memory once, and the waves are long enough for the chip not to be bound by starting
// them.  The two divisions a lane needs are multiplications by rounded-up reciprocals: c = l / ng
// (exact for l < 2^32 / ng, and l < 64 E < 2^19) and group = rank / per (rank < 64).
constexpr int kBuildRows = 4;
__global__ __launch_bounds__(kSwapThreads) void swap_build_kernel(SwapParams p) {
  int cut = 0, block = blockIdx.x;
  while (cut + 1 < p.ncuts && block >= p.build_blocks[cut]) block -= p.build_blocks[cut++];
  const int ng = p.ng[cut], r0 = blockIdx.y * kBuildRows;
  const int l = block * kSwapThreads + threadIdx.x;
  if (l >= p.E * ng) return;
  const int32_t *__restrict__ const C = p.C[cut];
  const int32_t *__restrict__ const CG = p.CG[cut];
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
      int cba = 0;
#pragma unroll 8
      for (int k = 0; k < p.copies; ++k) cba += C[((int64_t)k * p.E + b) * p.E + a];
      add[i] = L0[a] - CG[(int64_t)a * ng + j];
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
// Bytes of LDS for the terms of the pairs, and for staged counts what is left of the 64 KiB that every launch gets.
constexpr int kSelectTerms = kMaxDim * kSelectPairs * (int)sizeof(double), kSelectStaged = 65536 - kSelectTerms;

struct SelectParams {
  int32_t d, G, E;
  int32_t U[kMaxDim];
  double M, v, gamma;
  const int32_t *z_inter[kMaxDim];
  const int32_t *z_intra;
  double scale_inter[kMaxDim], alpha_inter[kMaxDim], beta_inter[kMaxDim];
  double scale_intra, alpha_intra, beta_intra;
  double fan[kMaxDim];      // of term i: U[i + 1] / U[i], G / U[d - 1] of the last
  int32_t tile[kMaxDim];    // where the counts of term i are staged in LDS, in 16 bytes; -1: they are not
  double *Q;
  double *block_min;    // workspace [nblocks]
  int32_t *block_arg;   // workspace [nblocks]
  int32_t nblocks;
  int32_t *best_pair;
  double *best_time;
};

// x[0 .. N) of a term's counts, 0 beyond n <= N (counts are >= 0, so the padding changes neither the maximum
// nor, skipped, the sum).  Every load unconditional (the last count again beyond n), so that none waits for another.
template <int N>
__device__ __forceinline__ void load_counts(const int32_t *x, int n, int (&v)[N]) {
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

// The same for whole fours, through LDS: a lane that reads its pair's counts from memory touches a line of its own, so
// a wave's load is 64 lines, and a CU's cache holds the lines of few waves.  It pays where lanes read up to 64 counts
// (256 experts, terms of 8, 16, 32 and 64 groups, the whole selection 16.0 -> 14.3 us; of 4, 8, 16 and 32 11.0 from
// memory, 11.3 so; 512 experts 23.8, 25.7).  The wave takes its 64 pairs in order, straight into LDS (`tile`, 256 n
// bytes), `first` its first four of the `fours` there are in all.  Within the fours of a pair, if they are a power of
// two, the places are exchanged from pair to pair, so that the lanes, which then read one pair each, spread over all
// banks.
template <int N>
__device__ __forceinline__ void stage_counts(i32x4 *tile, const i32x4 *z, int64_t first, int64_t fours, int n, int (&v)[N]) {
  const int lane = lane_id(), nq = n >> 2, log2_nq = 31 - __builtin_clz(nq);
  const int mask = (nq & (nq - 1)) == 0 && nq <= 16 ? nq - 1 : 0, shift = mask ? 4 - log2_nq : 0;
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    if (i >= nq) break;
    const int slot = i * kWave + lane, pair = mask ? slot >> log2_nq : 0;
    const int64_t four = min(first + (slot ^ ((pair >> shift) & mask)), fours - 1);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(z + four),
                                     (__attribute__((address_space(3))) void *)(tile + i * kWave), 16, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the wave's own loads are in LDS
  __asm__ volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    const i32x4 w = tile[lane * nq + (min(i, nq - 1) ^ ((lane >> shift) & mask))];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * i + e] = i < nq ? w[e] : 0;
  }
}

// The smooth maximum of Eq.(11) of n <= N counts x, which v holds.  Every lane is a chain of fp64 operations and there
// is about one wave per SIMD, so the chain is what counts: a whole gamma is raised for eight counts
// side by side, one pass over its bits for all of them; the sum itself stays in the order of the
// counts.
template <int N>
__device__ __forceinline__ double smooth_max(const int (&v)[N], const int32_t *x, int n, double gamma) {
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
    for (int j = 0; j < n; ++j) sum += pow((double)x[j] / m, gamma);
  }
  return m * pow(sum, 1.0 / gamma);
}

__device__ __forceinline__ void keep_better(double &val, int32_t &arg, double v, int32_t a) {
  const bool better = a >= 0 && (arg < 0 || v < val || (v == val && a < arg));   // among equal times the lower pair index
  val = better ? v : val;
  arg = better ? a : arg;
}
// The words of the lane `OFF` away (OFF a power of two): within rows of sixteen by the data paths of the vector unit,
// across them by swaps of rows.  (Through LDS, as shuffles, the six steps of an argmin wait for three trips each.)
template <int OFF>
__device__ __forceinline__ uint32_t from_lane(uint32_t v) {
  if constexpr (OFF == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return lane_id() & 32 ? r[0] : r[1];
  } else if constexpr (OFF == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return lane_id() & 16 ? r[0] : r[1];
  } else {   // by 8; 7 - i within eight lanes, which are alike in pairs of four by then; quads
    constexpr int kControl = OFF == 8 ? 0x128 : OFF == 4 ? 0x141 : OFF == 2 ? 0x4E : 0xB1;
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kControl, 0xF, 0xF, true);
  }
}
template <int OFF>
__device__ __forceinline__ void argmin_step(double &val, int32_t &arg) {
  const uint64_t bits = __builtin_bit_cast(uint64_t, val);
  const uint64_t other = (uint64_t)from_lane<OFF>((uint32_t)(bits >> 32)) << 32 | from_lane<OFF>((uint32_t)bits);
  keep_better(val, arg, __builtin_bit_cast(double, other), (int32_t)from_lane<OFF>((uint32_t)arg));
}
__device__ __forceinline__ void wave_argmin(double &val, int32_t &arg) {
  argmin_step<32>(val, arg);
  argmin_step<16>(val, arg);
  argmin_step<8>(val, arg);
  argmin_step<4>(val, arg);
  argmin_step<2>(val, arg);
  argmin_step<1>(val, arg);
}

// Q of 64 pairs by a workgroup: a wave per term of Eq.(8) (the Inter levels 1 .. d-1, then the Intra level), a lane per
// pair, so that the waves with few groups are done early instead of waiting for the lanes of the widest cut, and
// everything about a term is uniform.  Neighbouring workgroups begin with another term, so that the widest ones do not
// meet on one SIMD.  The terms are then added in the order of the levels, so Q has the bits of a serial evaluation.
// The whole selection (graphs of twenty), every workgroup beginning with the first term and argmins by shuffles -> now:
// 128 experts 8.9 -> 8.5 us, 256 11.7 -> 11.0.  Tried: the root by one step of Halley's method from a guess in binary32
// (0.3 and 0.7 us less, but one Q in 25 differs in the last bit, which decides between pairs of equal time).
template <int N>   // most groups of a term: 32 or 64
__global__ __launch_bounds__(kSelectThreads) void swap_q_kernel(SelectParams p) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) i32x4 count_tiles[];
  __shared__ double s_term[kMaxDim][kSelectPairs];
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int term = (w + (int)blockIdx.x) & (kMaxDim - 1);
  const int64_t rc = (int64_t)blockIdx.x * kSelectPairs + lane, pairs = (int64_t)p.E * p.E;
  const bool live = rc < pairs;
  if (term < p.d) {
    const bool intra = term == p.d - 1;
    const int i = intra ? 0 : term + 1;
    const int n = intra ? p.G : p.U[i];
    const int32_t *const z = intra ? p.z_intra : p.z_inter[i];
    const double fan = p.fan[term];
    const double scale = intra ? p.scale_intra : p.scale_inter[i];
    const double beta = intra ? p.beta_intra : p.beta_inter[i], alpha = intra ? p.alpha_intra : p.alpha_inter[i];
    const int32_t *const x = z + (live ? rc : 0) * n;
    int v[N];
    if (N > 32 && p.tile[term] >= 0)
      stage_counts<N>(count_tiles + p.tile[term], (const i32x4 *)z, (int64_t)blockIdx.x * (kSelectPairs / 4) * n, pairs * (n >> 2), n, v);
    else
      load_counts<N>(x, n, v);
    const double volume = fan * scale * smooth_max<N>(v, x, n, p.gamma) * p.M * p.v;
    s_term[term][lane] = volume * beta + alpha;
  }
  __syncthreads();
  if (w != 0) return;
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
// one value: four minima per lane in flight, then steps within the waves and one across them.
constexpr int kArgminThreads = 1024, kArgminFew = 256;   // lanes; for up to four minima each of the few
template <int THREADS>
__global__ __launch_bounds__(THREADS) void swap_argmin_kernel(SelectParams p) {
  constexpr int kWaves = THREADS / kWave;
  __shared__ double s_val[kWaves];
  __shared__ int32_t s_arg[kWaves];
  double best = 0.0;
  int32_t arg = -1;
  for (int b0 = 0; b0 < p.nblocks; b0 += 4 * THREADS) {
    double v[4];
    int32_t a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int b = b0 + j * THREADS + (int)threadIdx.x;
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

// Whether the workspace has partial tables of chunks (and a byte per slot): E <= 256 and chunks short enough for
// 16-bit counts.
static inline bool swap_has_parts(int64_t E, int64_t T) { return E <= kCoocPartMaxE && T <= (int64_t)kCoocChunks * kCoocChunkTokensMax; }
// Private copies of C on the path with atomics: as many as fit 2 MiB per cut, at most
// kSwapCopiesMax (32 for E <= 128, 8 for E = 256): more copies spread the atomics of popular pairs,
// but each is cleared and summed again.  One where there are partial tables, which the atomics only stand in for.
static inline int64_t swap_copies(int64_t E, int64_t T) {
  if (swap_has_parts(E, T)) return 1;
  int64_t n = kSwapCopiesMax;   // a power of two, so that a workgroup finds its copy with a mask
  while (n > 1 && n * E * E > (int64_t)(1 << 19)) n /= 2;
  return n;
}

// Workspace, in ints: L0 [E], then per cut base [64] | L [E] | CG [E * ng] | C [copies * E * E], and where there are
// parts room for those of kCoocChunks chunks and for another C and CG.  The sizes are a promise to callers who keep such
// a buffer.  The matrix path needs less, the tables of its chunks: it lays them out over all of it, cut after cut.
static inline int64_t cooc_part_words(int64_t E, int64_t ng) { return (E * E + E * ng + 65) / 2; }
static inline int64_t swap_cut_ints(int64_t E, int64_t ng, int64_t T) {
  return 64 + E + E * ng + swap_copies(E, T) * E * E +
         (swap_has_parts(E, T) ? kCoocChunks * cooc_part_words(E, ng) + E * E + E * ng : 0);
}
// ... and, on the matrix path, one byte per routing slot at the very end.
static inline int64_t swap_slot_ints(int64_t T, int64_t K, int64_t E) { return swap_has_parts(E, T) ? (T * K + 3) / 4 : 0; }

// The matrix kernel for E experts, the columns of a panel, the tokens of a tile (0: the device does not grant the LDS).
typedef void (*cooc_kernel_t)(CoocParams);
struct CoocLaunch {
  cooc_kernel_t kernel;
  int panel, tile_tokens, stride;
  size_t lds;
};
template <int COLS, bool OWN_SLOTS, bool ADDED>
static CoocLaunch cooc_launch(int E, int groups, int64_t tokens) {   // groups of the finest cut, tokens of a chunk
  static const bool granted = [] {
    const hipError_t e = hipFuncSetAttribute((const void *)swap_cooc_kernel<COLS, OWN_SLOTS, ADDED>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kCoocLds);
    if (e != hipSuccess) (void)hipGetLastError();   // not sticky: do not let it fail the next launch check
    return e == hipSuccess;
  }();
  constexpr int kBatch = 4 / COLS * kCoocStep;   // a tile is whole batches of products
  const int rows = CoocTiles<COLS>(E, groups).rows();
  int most = 2 * (kCoocLds / rows - kCoocPad) / kBatch * kBatch;
  if (most > kCoocThreads) most = kCoocThreads;
  CoocLaunch l = {swap_cooc_kernel<COLS, OWN_SLOTS, ADDED>, 32 * COLS, 0, 0, 0};
  if (!granted) return l;
  const int64_t tiles = tokens > most ? (tokens + most - 1) / most : 1;   // all of a size
  l.tile_tokens = (int)(((tokens + tiles - 1) / tiles + kBatch - 1) / kBatch * kBatch);
  if (l.tile_tokens < kBatch) l.tile_tokens = kBatch;   // no tokens at all
  l.stride = l.tile_tokens / 2 + kCoocPad;
  l.lds = (size_t)rows * l.stride;
  return l;
}
template <int COLS>
static inline CoocLaunch cooc_launch_for(int E, bool own_slots, bool parts, int groups, int64_t tokens) {
  if (!parts) return cooc_launch<COLS, true, true>(E, groups, tokens);
  return own_slots ? cooc_launch<COLS, true, false>(E, groups, tokens) : cooc_launch<COLS, false, false>(E, groups, tokens);
}
static inline int cooc_chunks(bool parts, int64_t T, int64_t E, int ncuts) {
  if (parts) return kCoocChunks;
  const int64_t panel = 32 * cooc_columns((int)E), panels = (E + panel - 1) / panel, tiles = (T + 127) / 128;
  const int64_t most = kCoocAddedGroups / (panels * ncuts), least = (T + kCoocAddedTokensMax - 1) / kCoocAddedTokensMax;
  const int64_t chunks = most > tiles ? tiles : most;
  return (int)(chunks < least ? least : chunks < 1 ? 1 : chunks);
}

// Whether atomics per slot are faster than matrix products whose chunks are added up: with few slots per token or few
// groups, as the products take the same time however few marks a tile holds.  Two straight lines, us, through some
// 4,000 shapes (256 < E <= 512, up to 520,000 tokens; E <= 256, 522,241 to 800,000; one to eight slots, one to four
// cuts; ids drawn evenly): Z, the updates of C (a slot's K - 1 others where it is alone in its group) and of L0, L and
// CG (in LDS or in memory), and the workgroups that put their tables together; against Z and a time per tile, for its
// barriers, its tokens and the bytes cleared (within 10 % for nine in ten).  A popular few experts make only the
// atomics slower, and those of C most, so they have to be ahead by a tenth if there are such; without (one slot, or one
// group) they may be estimated behind by an eighth, by which the line for them is too high there.  Of 1,500 shapes,
// half of them with a Zipf router, the rule loses more than 3 % in 122 (95 Zipf ids by atomics). Atomics / matrices: E
// = 320, one group, 18,696 tokens, K = 1 11.2 / 15.9; E = 288, 46,004 tokens, cuts of 1 and 8, K = 2 23 / 30; E = 512,
// cuts of 16 and 64, 373,641 tokens, K = 2, Zipf 4,663 / 399; E = 64, one group, 700,000 tokens, K = 2 24 / 45.
static bool atomics_pay(int64_t T, int64_t K, int64_t E, int ncuts, const int32_t *ng, bool in_lds, int64_t tiles, const CoocLaunch &cooc) {
  double groups = 0.0, others = 0.0, touched = 1.0;   // per slot: updates of C, words of L0, L and CG
  for (int c = 0; c < ncuts; ++c) {
    double alone = (double)(K - 1);
    for (int64_t k = 1; k < K; ++k) alone *= 1.0 - 1.0 / ng[c];
    groups += ng[c];
    others += alone;
    touched += 1.0 + (double)(K < ng[c] ? K : ng[c]);
  }
  int64_t lanes = 1;
  while (lanes < K) lanes *= 2;
  const double pairs = (double)(E * E) * 1e-6, slots = (double)(T * K) * 1e-6, filled = (double)(T * lanes) / (256.0 * kFactorThreads);
  const double flush = filled < 1.0 ? filled : 1.0;   // of 256 workgroups
  const double atomics = in_lds ? 10.0 + 4.3 * pairs * groups + slots * (28.0 * others + 1.4 * touched) + 3.2 * ncuts + 6.6 * flush
                                : 45.0 + 2.4 * pairs * groups + 54.0 * slots * touched + 59.0 * flush;
  const double tile = 0.4 + 0.0019 * cooc.tile_tokens + 0.175 * (double)cooc.lds / 16384.0;
  const double matrices = 9.7 + 6.3 * pairs * ncuts + 0.7 * pairs * groups + (double)tiles * tile;
  return (others < 0.05 ? 0.85 : 1.1) * atomics < matrices;
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
  if (parts || (own_slots && E <= kCoocMaxE)) {   // parts imply E <= 256
    CoocParams cp;
    int groups = 1;
    for (int c = 0; c < ncuts; ++c) groups = ng[c] > groups ? ng[c] : groups;
    cp.chunks = cooc_chunks(parts, T, E, ncuts);
    const int64_t steps = ((int64_t)T + kCoocStep - 1) / kCoocStep;
    cp.tokens_per_chunk = (int32_t)((steps + cp.chunks - 1) / cp.chunks * kCoocStep);
    const CoocLaunch cooc = cooc_columns(E) == 2 ? cooc_launch_for<2>(E, own_slots, parts, groups, cp.tokens_per_chunk)
                                                   : cooc_launch_for<1>(E, own_slots, parts, groups, cp.tokens_per_chunk);
    const int tiles = cooc.lds ? (cp.tokens_per_chunk + cooc.tile_tokens - 1) / cooc.tile_tokens : 0;
    if (cooc.lds != 0 && (parts || !atomics_pay(T, K, E, ncuts, ng, in_lds, tiles, cooc))) {
      PairParams pp;
      cp.ids = topk_ids;
      cp.expert_to_rank = expert_to_rank;
      cp.T = T;
      cp.K = K;
      cp.E = E;
      cp.G = G;
      cp.ncuts = ncuts;
      cp.sub_log2 = 0;
      while ((1 << cp.sub_log2) < K) ++cp.sub_log2;
      cp.k_reciprocal = K > 1 ? (uint32_t)((0x100000000ull + (uint64_t)K - 1) / (uint64_t)K) : 0u;
      cp.tile_tokens = cooc.tile_tokens;
      cp.stride = cooc.stride;
      cp.words_recip17 = (uint32_t)((1 << 17) + cooc.tile_tokens / 8 - 1) / (uint32_t)(cooc.tile_tokens / 8);
      cp.slot_bits = (uint8_t *)(p.ws + at);
      cp.status = status;
      int64_t tables = 0;   // they take less room than a cut has for its tables by atomics, or its parts
      for (int c = 0; c < kMaxCuts; ++c) {
        const int cc = c < ncuts ? c : 0;
        cp.ng[c] = p.ng[cc];
        cp.per[c] = p.per[cc];
        cp.per_recip16[c] = (uint32_t)((65536 + cp.per[c] - 1) / cp.per[c]);
        cp.tables[c] = c < ncuts ? p.ws + tables : cp.tables[0];
        if (c < ncuts) tables += parts ? (Tables::values(E, ng[c]) * cp.chunks + 1) / 2 : Tables::values(E, ng[c]);
        PairCut &cut = pp.cut[c];
        cut.tables = cp.tables[c];
        cut.Z = p.Z[cc];
        cut.ng = cp.ng[c];
        cut.per_recip16 = cp.per_recip16[c];
        cut.wide = cut.ng % 4 == 0 ? 4 : 1;
        cut.of_pair = cut.ng / cut.wide;
        cut.of_pair_recip20 = ((1 << 20) + cut.of_pair - 1) / cut.of_pair;
        cut.pairs_at_once = kPairThreads / cut.of_pair;
      }
      p.ws_ints = parts ? 0 : tables;   // parts are written in full: only the status word needs clearing
      if (status || p.ws_ints) {
        const int64_t n = p.ws_ints > 0 ? p.ws_ints : 1;
        hipLaunchKernelGGL(swap_clear_kernel, dim3((unsigned)((n + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads), 0, stream, p);
        if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
      }
      if (T > 0 && !own_slots) {
        const int64_t lanes = (int64_t)T << cp.sub_log2;
        hipLaunchKernelGGL(swap_slots_kernel, dim3((unsigned)((lanes + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads), 0,
                           stream, cp);
        if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
      }
      const int panels = (E + cooc.panel - 1) / cooc.panel;
      hipLaunchKernelGGL(cooc.kernel, dim3((unsigned)cp.chunks, (unsigned)ncuts, (unsigned)panels), dim3(kCoocThreads), cooc.lds, stream, cp);
      if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
      pp.expert_to_rank = expert_to_rank;
      pp.E = E;
      pp.G = G;
      pp.ncuts = ncuts;
      pp.blocks = (E + kBlock - 1) / kBlock;
      pp.status = status;
      const unsigned blocks = (unsigned)pp.blocks;
      hipLaunchKernelGGL((!parts ? swap_pairs_kernel<int32_t, 1> : swap_pairs_kernel<uint16_t, kCoocChunks>),
                         dim3(blocks, blocks / 2 + 1, (unsigned)ncuts), dim3(kPairThreads), 0, stream, pp);
      return hm_launch_status();
    }
  }
  p.ws_ints = at;
  p.use_lds = in_lds ? 1 : 0;
  hipLaunchKernelGGL(swap_clear_kernel, dim3((unsigned)((p.ws_ints + kSwapThreads - 1) / kSwapThreads)), dim3(kSwapThreads), 0, stream,
                     p);
  if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  if (T > 0) {
    const int64_t tokens_per_block = (int64_t)(kFactorThreads / kWave) * (kWave / p.sub);
    int64_t blocks = ((int64_t)T + tokens_per_block - 1) / tokens_per_block;
    if (blocks > 256) blocks = 256;   // one per CU; every block flushes its LDS tables with atomics
    hipLaunchKernelGGL(swap_factors_kernel, dim3((unsigned)blocks), dim3(kFactorThreads), p.use_lds ? (size_t)lds_at * sizeof(int32_t) : 0,
                       stream, p);
    if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  }
  int64_t build_blocks = 0;
  for (int c = 0; c < kMaxCuts; ++c) {
    p.build_blocks[c] = c < ncuts ? (int32_t)(((int64_t)E * p.ng[c] + kSwapThreads - 1) / kSwapThreads) : 0;
    build_blocks += p.build_blocks[c];
  }
  hipLaunchKernelGGL(swap_build_kernel, dim3((unsigned)build_blocks, (unsigned)((E + kBuildRows - 1) / kBuildRows)), dim3(kSwapThreads), 0,
                     stream, p);
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
  int fours = 0;
  for (int i = 0; i < kMaxDim; ++i) {
    const bool intra = i == d - 1;
    const int n = intra ? G : i < d ? U[i + 1] : 1;
    const int32_t *const z = intra ? z_intra : i < d ? z_inter[i + 1] : nullptr;
    p.fan[i] = intra ? (double)(G / U[d - 1]) : i < d ? (double)(U[i + 1] / U[i]) : 0.0;
    // The loads into LDS are of 16 bytes.  Four terms of 64 groups (U = 1, 64, 64, 64) do not all fit: the last is read
    // from memory.
    const int more = kSelectPairs * n / 4;
    const bool staged = i < d && G > 32 && n % 4 == 0 && ((uintptr_t)z & 15) == 0 && 16 * (fours + more) <= kSelectStaged;
    p.tile[i] = staged ? fours : -1;
    if (staged) fours += more;
  }
  hipLaunchKernelGGL(G <= 32 ? swap_q_kernel<32> : swap_q_kernel<64>, dim3(p.nblocks), dim3(kSelectThreads), (size_t)fours * 16, stream, p);
  if (hm_launch_status() != HM_OK) return HM_ERR_HIP;
  if (p.nblocks <= 4 * kArgminFew) hipLaunchKernelGGL(swap_argmin_kernel<kArgminFew>, dim3(1), dim3(kArgminFew), 0, stream, p);
  else hipLaunchKernelGGL(swap_argmin_kernel<kArgminThreads>, dim3(1), dim3(kArgminThreads), 0, stream, p);
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
