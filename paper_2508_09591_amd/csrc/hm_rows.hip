// Row-streaming kernels: hm_dispatch_pack, hm_combine, hm_combine_transpose.
//
// All three are HBM-bound and token-centric: a wave owns (token, segment of the row), reads the
// token-side data once and touches each of the token's distinct packed rows once, which is the
// algorithmic minimum of (1 + c) rows of traffic per token (c = packed rows per token).  The
// token's row list is wave-uniform: lanes 0..K-1 fetch slot_row[t,:], a ballot marks the rows to
// visit and readlane broadcasts each row index into a scalar register, so every global access
// is a base + lane*16 B coalesced stream of 16-byte vectors.
//
// Segments are 64 consecutive 16-byte vectors (1 KiB, one vector per lane).  Work items this
// small matter on MI355X: a kernel here lasts well under 100 us on the DeepSeek-V3 shape, so with
// multi-KiB items the last round of waves leaves most of the chip idle.  Every row-sized stream
// is read and written with non-temporal accesses: rows are touched once per kernel, and output
// lines left dirty in the caches were measured to slow the next kernel down by about 10 %.
//
// Waves per CU are capped on purpose.  With every wave slot filled, a kernel that writes (or
// reads) seven or eight 1 KiB pieces per wave has several hundred KiB per CU queued at the
// memory system, and the rate drops (a flat 1-read + 7-write stream: 64 % of peak with 32 waves
// per CU, 78 % with 8); with too few waves the index lookups are no longer hidden.  The cap is
// set with an unused dynamic LDS allocation: dispatch runs 24 waves per CU (-5 % on the 64 Ki-token
// layer at node level, -9 % at rank level, neutral elsewhere), or 12 where many rows per token meet
// cached tokens; the bf16 transpose does more arithmetic per byte and is faster uncapped, the fp32 one is
// capped where transpose_capped says so; combine keeps about 128 KiB of row loads in flight per CU (32 waves
// up to four rows per token, 16 at eight).
//
// That is the form for rows of whole 128-byte lines that are wider than a wave's lanes.  Rows that begin inside a
// line, of any length, narrow, odd or few have forms of their own: spread_route and combine_route, at the end, say
// which call takes which, and the kernels say what each is bound by.
//
// Combine has two forms.  With the caller's weights (topk_weights != NULL) every wave finds the rows of its
// token and merges its K slots itself (3K readlanes), the weights behind the first loads.  With the plan's
// merged weights (topk_weights == NULL) the first slot of each row is the one slot_keep marks and its
// weight is one gathered load from row_weight: 1 to 3 % faster.  A wave takes 1 KiB of the row with all of
// the token's rows (up to eight) in flight, with the caller's weights where short_segments says so, else 4 KiB.
// Tokens with about one row each (the local-expert stage of a receiver) keep 4 KiB segments, two
// rows in flight: a 1 KiB segment would be mostly prologue there (0.36 vs 0.28 ms on that stage).
#include "hm_device.h"

#include <atomic>
#include <type_traits>

namespace hm {

constexpr int kElemThreads = 256;     // element-wise fallback kernels
constexpr int kCopyThreads = 128;     // dispatch / transpose: two waves per workgroup ...
constexpr int kCopyWavesPerCu = 24;   // ... and this many waves resident per CU, where they are capped
constexpr int kCombineThreads = 256;
constexpr int kCombineVecs = 4;       // combine of tokens with few rows, or an unknown number: 16-byte vectors per lane (4 KiB segments),
constexpr int kCombineRows = 4;       //   rows whose loads are in flight together
constexpr int kCombineRowsFew = 2;    //   ... or two, when the tokens are known to have fewer than two rows
constexpr int kCombineRowsPlan = 8;   // combine, 1 KiB segments (two rows per token or more):
                                      //   up to eight rows in flight
constexpr int kCombineBytesInFlight = 128 * 1024;   // per CU, what the cap on resident waves aims at

constexpr int kLineBytes = 128;
constexpr int32_t kMaxVectorH = 1 << 30;   // the vector kernels count elements of a row in 32 bits

struct RowParams {
  int32_t T, K;
  int32_t H;      // elements per row
  int32_t nvec;   // 16-byte vectors per row (whole rows)
  int32_t shift;  // elements between a 128-byte line and the start of the buffer written (ragged rows)
  int32_t nseg;   // segments per row
  int64_t nunits; // T * nseg (flat kernels: T * nvec)
  uint64_t recip; // ceil(2^64 / nseg) (flat kernels: / nvec), 0 for 1
  const int32_t *slot_row;
  const uint8_t *slot_keep;
  int32_t *status;
};

// n / d for the reciprocal ceil(2^64 / d) (0 for d = 1): exact while n d < 2^64.
__device__ __forceinline__ int64_t divided(int64_t n, uint64_t recip) {
  return recip ? (int64_t)__umul64hi((uint64_t)n, recip) : n;
}

// The workgroup's place among the others: as launched, or (NEAR) in groups of 128 neighbours that run on one die, the
// groups going round the dies; a short last round is as launched.  Workgroups go round the eight dies, and each die has
// an L2 of its own: where rows begin inside a line, the line that two workgroups share is written from two dies, twice
// and in part.  Those lines are what ragged rows lose: 4,097 x 1,030, six rows per token, dispatch 15.2 us, 11.8 when
// the shared lines are left out, 14.3 grouped; 15.2 -> 19.5 when they are written through the caches.  Counters of that
// layer, as launched -> grouped: 791,000 write requests to memory both ways, those of less than 64 bytes 21,200 ->
// 8,700; bytes read, as neighbours share the lines they read too, 1.25 -> 1.02 times the tokens'.  near_pays() says
// where the grouping is used.
constexpr unsigned kDies = 8, kNear = 128;
template <bool NEAR>
__device__ __forceinline__ unsigned block_place() {
  if constexpr (!NEAR) return blockIdx.x;
  constexpr unsigned round = kDies * kNear;
  const unsigned b = blockIdx.x, in = b % round, first = b - in;
  return first + round <= gridDim.x ? first + in % kDies * kNear + in / kDies : b;
}

// Wave-uniform (token, segment) of this wave, or false when past the end.
template <int BLOCK, bool DIVIDE = false, bool NEAR = false>
__device__ __forceinline__ bool unit_of_wave(const RowParams &p, int &t, int &seg) {
  const int64_t unit = (int64_t)block_place<NEAR>() * (BLOCK / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (unit >= p.nunits) return false;
  t = (int)(DIVIDE ? unit / p.nseg : divided(unit, p.recip));
  seg = (int)(unit - (int64_t)t * p.nseg);
  return true;
}

// How a row is cut into 16-byte vectors.
// WholeRows: the rows of both buffers are whole, aligned 16-byte vectors; vector v is elements [v P, v P + P).
// RaggedRows: any length of at least one vector, at the alignment of the elements.  The vectors follow
// the 16-byte grid of the buffer that is WRITTEN, counted from the 128-byte line that holds the row's
// first element, so that two waves share no line inside a row: a wave that stores part of a line
// leaves the rest to a wave behind another die's L2, and each of them then writes a piece of it to
// memory.  Reads take whatever alignment results.  A vector that reaches over the row's first or last
// element is moved inside the row instead: its values are computed twice from the same inputs, to the same
// bits, and stored twice, which needs neither a tail loop nor a mask.  (Where the last vector is the first
// of a wave's segment, that wave stores into the last line of the wave before it, too.)
template <typename ELEM>
struct WholeRows {
  typedef u32x4 vec;
  static __device__ __forceinline__ bool place(const RowParams &p, int64_t, int v, int &at) {
    at = v * (int)(16 / sizeof(ELEM));
    return v < p.nvec;
  }
};
template <typename ELEM>
struct RaggedRows {
  typedef std::conditional_t<sizeof(ELEM) == 2, u32x4_align2, u32x4_align4> vec;
  // Vector v of the row as it lies in the buffer written: its first element, false if it is outside the row.
  static __device__ __forceinline__ bool place(const RowParams &p, int64_t row, int v, int &at) {
    constexpr int P = 16 / sizeof(ELEM), kLine = kLineBytes / sizeof(ELEM);
    const int before = (int)((uint32_t)row * (uint32_t)p.H + (uint32_t)p.shift) & (kLine - 1);
    const int e = v * P - before;
    at = min(max(e, 0), p.H - P);
    return e > -P && e < p.H;
  }
};
template <typename ACCESS, typename ELEM>
__device__ __forceinline__ u32x4 load_row(const ELEM *base, const RowParams &p, int64_t row, int at) {
  return __builtin_nontemporal_load((const typename ACCESS::vec *)(base + (row * p.H + at)));
}
template <typename ACCESS, typename ELEM>
__device__ __forceinline__ void store_row(ELEM *base, const RowParams &p, int64_t row, int at, u32x4 value) {
  __builtin_nontemporal_store(value, (typename ACCESS::vec *)(base + (row * p.H + at)));
}

// ---------------------------------------------------------------------------------------------
// dispatch: packed[slot_row[t,k], :] = x[t, :] for kept slots
// ---------------------------------------------------------------------------------------------
template <bool NEAR>
__global__ __launch_bounds__(kCopyThreads) void dispatch_rows_kernel(RowParams p, const uint16_t *__restrict__ x,
                                                                     uint16_t *__restrict__ packed, int64_t packed_rows) {
  int t, seg;
  if (!unit_of_wave<kCopyThreads, false, NEAR>(p, t, seg)) return;
  const int lane = lane_id();
  int at;
  const bool in_row = WholeRows<uint16_t>::place(p, 0, seg * kWave + lane, at);
  u32x4 r = {0u, 0u, 0u, 0u};
  if (in_row) r = *(const u32x4 *)(x + ((int64_t)t * p.H + at));   // does not wait for the row list below
  int my_row = -1;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    if (p.slot_keep[s] && row >= 0) {
      if (row < packed_rows) my_row = row;
      else if (seg == 0) flag(p.status, HM_ERR_CAPACITY);
    }
  }
  uint64_t todo = __ballot(my_row >= 0);
  while (todo) {
    const int k = __builtin_ctzll(todo);
    todo &= todo - 1;
    const int row = read_lane(my_row, k);
    if (in_row) store_row<WholeRows<uint16_t>>(packed, p, row, at, r);
  }
}

// Any H / any alignment: one thread per (token, element), 2-byte accesses.
__global__ __launch_bounds__(kElemThreads) void dispatch_elems_kernel(RowParams p, int32_t H, const uint16_t *__restrict__ x,
                                                                     uint16_t *__restrict__ packed, int64_t packed_rows) {
  const int64_t i = (int64_t)blockIdx.x * kElemThreads + threadIdx.x;
  if (i >= (int64_t)p.T * H) return;
  const int t = (int)(i / H), j = (int)(i - (int64_t)t * H);
  const uint16_t v = x[i];
  for (int k = 0; k < p.K; ++k) {
    const int64_t s = (int64_t)t * p.K + k;
    const int row = p.slot_row[s];
    if (!p.slot_keep[s] || row < 0) continue;
    if (row < packed_rows) packed[(int64_t)row * H + j] = v;
    else if (j == 0) flag(p.status, HM_ERR_CAPACITY);
  }
}

// ---------------------------------------------------------------------------------------------
// combine: out[t,:] = bf16( sum over the token's distinct rows of (sum of their slots' weights) * y[row,:] )
// ---------------------------------------------------------------------------------------------
// Lane k < K holds slot k of the token.  On return `agg` is the fp32 sum, in ascending k, of the
// weights of all slots that share lane k's row, and the returned mask has bit k set for the
// lowest slot of each distinct valid row.
__device__ __forceinline__ uint64_t merge_slots(int K, int my_row, float my_w, float &agg) {
  const int lane = lane_id();
  agg = 0.0f;
  bool first = my_row >= 0;
  for (int k1 = 0; k1 < K; ++k1) {
    const int r1 = read_lane(my_row, k1);
    const float w1 = read_lane(my_w, k1);
    if (r1 == my_row && my_row >= 0) {
      agg = agg + w1;
      if (k1 < lane) first = false;
    }
  }
  return __ballot(first);
}

// Element type of a row as the combine kernels see it: how many values a 16-byte vector holds,
// how they enter the fp32 fma chain and how the fp32 sums are stored.
struct RowBf16 {
  typedef uint16_t elem;
  static constexpr int kPerVec = 8;
  static __device__ __forceinline__ void fma_into(float *acc, float a, u32x4 r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] = __builtin_fmaf(a, bf16_lo(r[e]), acc[2 * e]);
      acc[2 * e + 1] = __builtin_fmaf(a, bf16_hi(r[e]), acc[2 * e + 1]);
    }
  }
  static __device__ __forceinline__ u32x4 pack(const float *acc) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = pack_bf16x2(acc[2 * e], acc[2 * e + 1]);
    return o;
  }
  static __device__ __forceinline__ float widen(elem v) { return __builtin_bit_cast(float, (uint32_t)v << 16); }
  static __device__ __forceinline__ elem narrow(float f) { return (elem)f32_to_bf16(f); }
  // bf16(a * g) with ONE rounding.  The fp32 product p is already rounded; a second rounding to
  // bf16 differs from the exact one only when p sits exactly on a bf16 tie, and there the sign of
  // the product's rounding error e = fma(a, g, -p) says on which side the true value lies.  e is
  // exact as long as it does not underflow, i.e. for |a * g| >= 2^-102 or so; for smaller products
  // (gradients of that size do not occur in practice) a tie may be broken to even instead.
  static __device__ __forceinline__ uint32_t scale1(float a, float g) {
    const float p = a * g;
    const float e = __builtin_fmaf(a, g, -p);
    const uint32_t u = __builtin_bit_cast(uint32_t, p);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;   // NaN
    // round to nearest: add 0x7FFF plus a tie bit -- the kept lsb (ties to even) in general, but on
    // an exact tie of p with e != 0 the side the true product lies on
    const bool tie = (u & 0xFFFFu) == 0x8000u && e != 0.0f;
    const uint32_t away = ((__builtin_bit_cast(uint32_t, e) ^ u) >> 31) ^ 1u;   // e and p have the same sign
    const uint32_t tie_bit = tie ? away : ((u >> 16) & 1u);
    return (u + 0x7FFFu + tie_bit) >> 16;
  }
  static __device__ __forceinline__ elem scale(float a, elem g) { return (elem)scale1(a, widen(g)); }
  // Eight at once: the common path rounds the fp32 products to nearest even (add 0x7FFF plus the
  // kept lsb; the upper halves of two such sums are one output word, picked by a byte permute) and
  // only notes whether any product is a NaN or sits on a bf16 tie (1 in 65536); the exact
  // treatment runs for those vectors alone.
  static __device__ __forceinline__ u32x4 scale(float a, u32x4 r) {
    float g[8];
    uint32_t sum[8];
    bool special = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t w = r[e];
      g[2 * e] = bf16_lo(w);
      g[2 * e + 1] = bf16_hi(w);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float p = a * g[i];
      const uint32_t u = __builtin_bit_cast(uint32_t, p);
      sum[i] = u + 0x7FFFu + ((u >> 16) & 1u);
      special = special || (u & 0xFFFFu) == 0x8000u || __builtin_isnan(p);
    }
    u32x4 o;
    if (__builtin_expect(special, 0)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = scale1(a, g[2 * e]) | (scale1(a, g[2 * e + 1]) << 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_perm(sum[2 * e + 1], sum[2 * e], 0x07060302u);
    }
    return o;
  }
};
struct RowF32 {
  typedef float elem;
  static constexpr int kPerVec = 4;
  static __device__ __forceinline__ void fma_into(float *acc, float a, u32x4 r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t w = r[e];   // a copy first: a bit cast applied to the vector element itself reads element 0
      acc[e] = __builtin_fmaf(a, __builtin_bit_cast(float, w), acc[e]);
    }
  }
  static __device__ __forceinline__ u32x4 pack(const float *acc) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __builtin_bit_cast(uint32_t, acc[e]);
    return o;
  }
  static __device__ __forceinline__ float widen(elem v) { return v; }
  static __device__ __forceinline__ elem narrow(float f) { return f; }
  static __device__ __forceinline__ elem scale(float a, elem g) { return a * g; }   // one IEEE multiply
  static __device__ __forceinline__ u32x4 scale(float a, u32x4 r) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t w = r[e];
      o[e] = __builtin_bit_cast(uint32_t, a * __builtin_bit_cast(float, w));
    }
    return o;
  }
};

// MIX = false: hm_combine.  MIX = true: hm_combine_mix, the sum times the reciprocal of the sum of
// the merged weights (added in ascending k of each row's first slot); zero for a row without a
// valid slot.  (A true division per element made the kernel ALU-bound: 8 divisions per 16 bytes.)
template <bool MIX, int U, int R, typename ROW, typename ACCESS>
__global__ __launch_bounds__(kCombineThreads) void combine_rows_kernel(RowParams p, const typename ROW::elem *__restrict__ y,
                                                                       int64_t y_rows, const float *__restrict__ topk_weights,
                                                                       typename ROW::elem *__restrict__ out) {
  int t, seg;
  if (!unit_of_wave<kCombineThreads>(p, t, seg)) return;
  const int lane = lane_id();
  int my_row = -1;
  float my_w = 0.0f;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    if (row >= 0) {
      if (row < y_rows) {
        my_row = row;
        my_w = topk_weights[s];
      } else if (seg == 0) {
        flag(p.status, HM_ERR_CAPACITY);
      }
    }
  }
  float agg;
  uint64_t todo = merge_slots(p.K, my_row, my_w, agg);
  float inv_wsum = 0.0f;   // MIX: one division per wave, then a multiply per element
  if (MIX) {
    float wsum = 0.0f;
    for (uint64_t m = todo; m; m &= m - 1) wsum = wsum + read_lane(agg, __builtin_ctzll(m));
    inv_wsum = wsum != 0.0f ? 1.0f / wsum : 0.0f;
  }

  constexpr int E = ROW::kPerVec;
  int at[U];   // this lane's vectors: every 64th of the segment
  bool in_row[U];
#pragma unroll
  for (int i = 0; i < U; ++i) in_row[i] = ACCESS::place(p, t, seg * (kWave * U) + i * kWave + lane, at[i]);
  float acc[U][E];
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[i][e] = 0.0f;

  while (todo) {
    // issue the loads of up to R rows, then consume them in the same (ascending k) order
    u32x4 r[R][U];
    float a[R];
    bool have[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      have[j] = todo != 0;
      a[j] = 0.0f;
#pragma unroll
      for (int i = 0; i < U; ++i) r[j][i] = (u32x4){0u, 0u, 0u, 0u};
      if (have[j]) {
        const int k = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int row = read_lane(my_row, k);
        a[j] = read_lane(agg, k);
#pragma unroll
        for (int i = 0; i < U; ++i)
          if (in_row[i]) r[j][i] = load_row<ACCESS>(y, p, row, at[i]);
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (have[j]) {
#pragma unroll
        for (int i = 0; i < U; ++i) ROW::fma_into(acc[i], a[j], r[j][i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    if (in_row[i]) {
      if (MIX) {
#pragma unroll
        for (int e = 0; e < E; ++e) acc[i][e] = acc[i][e] * inv_wsum;
      }
      store_row<ACCESS>(out, p, t, at[i], ROW::pack(acc[i]));
    }
  }
}

// The same for tokens of two rows or more: a wave owns 1 KiB of the row, like combine_plan_rows_kernel, and goes by
// slots, eight at a time.  What bounds the call is the rows on their way, so a row's load is issued as soon as its slot
// is known to be the first with it, and the weights are merged behind the loads.  HIP events, three to sixteen pairs of
// buffers in turn, segments of 4 KiB with the weights first -> now (the plan's weights), us: 16,384 x 2,048 fp32 with 7
// rows 192 -> 183 (180), 8,192 x 7,168 with 3.1 rows 79.3 -> 75.9 (74.9), 8,192 x 2,048 with 7.4 49.9 -> 48.1 (47.6),
// 1,024 x 2,048 9.6 -> 8.2 (7.9), 256 x 4,096 7.7 -> 5.6 (5.3).
template <bool MIX, typename ROW, typename ACCESS>
__global__ __launch_bounds__(kCombineThreads) void combine_slots_kernel(RowParams p, const typename ROW::elem *__restrict__ y,
                                                                        int64_t y_rows, const float *__restrict__ topk_weights,
                                                                        typename ROW::elem *__restrict__ out) {
  constexpr int R = kCombineRowsPlan, E = ROW::kPerVec;
  int t, seg;
  if (!unit_of_wave<kCombineThreads>(p, t, seg)) return;
  const int lane = lane_id();
  int my_row = -1;
  float my_w = 0.0f;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    my_w = topk_weights[s];   // on its way with the row; not used where there is none
    if (row >= 0) {
      if (row < y_rows) my_row = row;
      else if (seg == 0) flag(p.status, HM_ERR_CAPACITY);
    }
  }
  int at;
  const bool in_row = ACCESS::place(p, t, seg * kWave + lane, at);
  float acc[E], agg = 0.0f, wsum = 0.0f;
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0f;
  for (int k0 = 0; k0 < p.K; k0 += R) {
    u32x4 r[R];
    bool first[R];   // slot k0 + j is the first of its row (uniform)
#pragma unroll
    for (int j = 0; j < R; ++j) {
      r[j] = (u32x4){0u, 0u, 0u, 0u};
      const int row = k0 + j < p.K ? read_lane(my_row, k0 + j) : -1;
      first[j] = row >= 0 && __builtin_ctzll(__ballot(my_row == row)) == k0 + j;
      if (first[j] && in_row) r[j] = load_row<ACCESS>(y, p, row, at);
    }
    if (k0 == 0) {   // the fp32 sum, in ascending k, of the weights of the slots that share lane k's row
      for (int k = 0; k < p.K; ++k) {
        const int row = read_lane(my_row, k);
        const float w = read_lane(my_w, k);
        if (row == my_row) agg = agg + w;
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (first[j]) {
        const float a = read_lane(agg, k0 + j);
        ROW::fma_into(acc, a, r[j]);
        wsum = wsum + a;
      }
    }
  }
  if (!in_row) return;
  if (MIX) {
    const float inv_wsum = wsum != 0.0f ? 1.0f / wsum : 0.0f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = acc[e] * inv_wsum;
  }
  store_row<ACCESS>(out, p, t, at, ROW::pack(acc));
}

// The same sum with the weights the plan merged: lane k < K holds slot k; the slot slot_keep marks
// is the first of its row, and row_weight[row] is the fp32 sum, in ascending k, of the weights of
// the slots that share the row -- the number merge_slots computes.  A wave owns U KiB of the row;
// the loads of up to R rows are issued before the first fma.
template <bool MIX, int U, int R, typename ROW, typename ACCESS>
__global__ __launch_bounds__(kCombineThreads) void combine_plan_rows_kernel(RowParams p, const typename ROW::elem *__restrict__ y,
                                                                            int64_t y_rows,
                                                                            const float *__restrict__ row_weight,
                                                                            typename ROW::elem *__restrict__ out) {
  int t, seg;
  if (!unit_of_wave<kCombineThreads>(p, t, seg)) return;
  const int lane = lane_id();
  int my_row = -1;
  float agg = 0.0f;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    if (p.slot_keep[s] && row >= 0) {
      if (row < y_rows) my_row = row;
      else if (seg == 0) flag(p.status, HM_ERR_CAPACITY);
    }
  }
  uint64_t todo = __ballot(my_row >= 0);
  if (my_row >= 0) agg = row_weight[my_row];   // in flight together with the first rows
  float inv_wsum = 0.0f;
  if (MIX) {
    float wsum = 0.0f;
    for (uint64_t m = todo; m; m &= m - 1) wsum = wsum + read_lane(agg, __builtin_ctzll(m));
    inv_wsum = wsum != 0.0f ? 1.0f / wsum : 0.0f;
  }
  constexpr int E = ROW::kPerVec;
  int at[U];   // this lane's vectors: every 64th of the segment
  bool in_row[U];
#pragma unroll
  for (int i = 0; i < U; ++i) in_row[i] = ACCESS::place(p, t, seg * (kWave * U) + i * kWave + lane, at[i]);
  float acc[U][E];
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[i][e] = 0.0f;
  while (todo) {
    u32x4 r[R][U];
    float a[R];
    bool have[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      have[j] = todo != 0;
      a[j] = 0.0f;
#pragma unroll
      for (int i = 0; i < U; ++i) r[j][i] = (u32x4){0u, 0u, 0u, 0u};
      if (have[j]) {
        const int k = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int row = read_lane(my_row, k);
        a[j] = read_lane(agg, k);
#pragma unroll
        for (int i = 0; i < U; ++i)
          if (in_row[i]) r[j][i] = load_row<ACCESS>(y, p, row, at[i]);
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (have[j]) {
#pragma unroll
        for (int i = 0; i < U; ++i) ROW::fma_into(acc[i], a[j], r[j][i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    if (in_row[i]) {
      if (MIX) {
#pragma unroll
        for (int e = 0; e < E; ++e) acc[i][e] = acc[i][e] * inv_wsum;
      }
      store_row<ACCESS>(out, p, t, at[i], ROW::pack(acc[i]));
    }
  }
}

// Any H / alignment: one thread per (token, element); same merge order and the same fma chain
// as the vector kernel, so both give identical bits.
template <bool MIX, typename ROW>
__global__ __launch_bounds__(kElemThreads) void combine_elems_kernel(RowParams p, int32_t H,
                                                                    const typename ROW::elem *__restrict__ y,
                                                                    int64_t y_rows, const float *__restrict__ topk_weights,
                                                                    const float *__restrict__ row_weight,
                                                                    typename ROW::elem *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kElemThreads + threadIdx.x;
  if (i >= (int64_t)p.T * H) return;
  const int t = (int)(i / H), j = (int)(i - (int64_t)t * H);
  const int32_t *rows = p.slot_row + (int64_t)t * p.K;
  float acc = 0.0f, wsum = 0.0f;
  for (int k = 0; k < p.K; ++k) {
    const int row = rows[k];
    if (row < 0) continue;
    bool first = true;
    for (int k1 = 0; k1 < k; ++k1) first = first && rows[k1] != row;
    if (!first) continue;
    if (row >= y_rows) {
      if (j == 0) flag(p.status, HM_ERR_CAPACITY);
      continue;
    }
    float agg = 0.0f;
    if (row_weight) {   // the plan's merged weight: the same additions in the same order
      agg = row_weight[row];
    } else {
      const float *w = topk_weights + (int64_t)t * p.K;
      for (int k1 = 0; k1 < p.K; ++k1)
        if (rows[k1] == row) agg = agg + w[k1];
    }
    acc = __builtin_fmaf(agg, ROW::widen(y[(int64_t)row * H + j]), acc);
    wsum = wsum + agg;
  }
  if (MIX) acc = acc * (wsum != 0.0f ? 1.0f / wsum : 0.0f);   // same reciprocal-multiply as the vector kernel
  out[i] = ROW::narrow(acc);
}

// ---------------------------------------------------------------------------------------------
// transpose: gy[slot_row[t,k], :] = row_weight[row] * gout[t, :] for kept slots (fp32)
// ---------------------------------------------------------------------------------------------
// DIVIDE: the wave's token by a division, which takes a wave some two hundred cycles longer than the multiplication
// everywhere else: bf16 rows of several GB are written faster by waves that start that much later (65,536 x
// 7,168, 7.5 rows per token: 1,437 us, 1,514 with the multiplication, 1,449 with it and a sleep of 512 cycles, 1,510
// with it and 24 waves per CU; 32,768 x 7,168 715 and 724, 65,536 x 4,096 with 7.3 rows 794 and 802; no
// difference below 2 GB), while with one row per token the multiplication is better (16,384 x 2,048 25.6 -> 24.9).
template <typename ROW, bool DIVIDE>
__global__ __launch_bounds__(kCopyThreads) void transpose_rows_kernel(RowParams p, const typename ROW::elem *__restrict__ gout,
                                                                      const float *__restrict__ row_weight,
                                                                      int64_t weight_rows, typename ROW::elem *__restrict__ gy,
                                                                      int64_t gy_rows) {
  typedef WholeRows<typename ROW::elem> access;
  int t, seg;
  if (!unit_of_wave<kCopyThreads, DIVIDE>(p, t, seg)) return;
  const int lane = lane_id();
  int at;
  const bool in_row = access::place(p, 0, seg * kWave + lane, at);
  u32x4 r = {0u, 0u, 0u, 0u};
  if (in_row) r = *(const u32x4 *)(gout + ((int64_t)t * p.H + at));
  int my_row = -1;
  float my_w = 0.0f;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    if (p.slot_keep[s] && row >= 0) {
      if (row < gy_rows && row < weight_rows) {
        my_row = row;
        my_w = row_weight[row];
      } else if (seg == 0) {
        flag(p.status, HM_ERR_CAPACITY);
      }
    }
  }
  uint64_t todo = __ballot(my_row >= 0);
  while (todo) {
    const int k = __builtin_ctzll(todo);
    todo &= todo - 1;
    const int row = read_lane(my_row, k);
    const float a = read_lane(my_w, k);
    if (in_row) store_row<access>(gy, p, row, at, ROW::scale(a, r));
  }
}

// Dispatch (SCALED = false: a bit copy) and transpose of ragged rows.  The rows written start at different places of a
// line, so the vectors of the token differ from row to row: each is read again, from the caches, at the place its row
// asks for; the reads of R rows are in flight together. Measured (8,192 / 16,384 tokens, bf16, HIP events, against
// vectors counted from the row's start): 7.3 copies of 2,051 elements 162 -> 123 us (4.5 TB/s), of 1,032 92 -> 76 us,
// of 7,160 251 -> 223 us; 3.6 copies of 4,140 68 -> 50 us.  Splitting a row evenly over its waves (no line grid) loses
// more than the last, short segment costs: 4,160 elements 218 -> 301 us; giving that segment to the wave before it
// changes nothing. R: rows whose reads are in flight together, eight where eight_reads_pay() says so, else four
// (dispatch and fp32: equal).  Tried: the wave's piece of the token in LDS, read once ahead of the row list, and each
// row's vectors from there (4,097 x 1,030, six rows: dispatch 15.2 -> 15.9, transpose 15.9 -> 16.8: the reads are not
// what it waits for).
template <typename ROW, bool SCALED, int R, bool NEAR>
__global__ __launch_bounds__(kCopyThreads) void spread_ragged_kernel(RowParams p, const typename ROW::elem *__restrict__ in,
                                                                     const float *__restrict__ row_weight, int64_t rows,
                                                                     typename ROW::elem *__restrict__ out) {
  typedef RaggedRows<typename ROW::elem> access;
  int t, seg;
  if (!unit_of_wave<kCopyThreads, false, NEAR>(p, t, seg)) return;
  const int lane = lane_id();
  int my_row = -1;
  float my_w = 0.0f;
  if (lane < p.K) {
    const int64_t s = (int64_t)t * p.K + lane;
    const int row = p.slot_row[s];
    if (p.slot_keep[s] && row >= 0) {
      if (row < rows) {
        my_row = row;
        if (SCALED) my_w = row_weight[row];
      } else if (seg == 0) {
        flag(p.status, HM_ERR_CAPACITY);
      }
    }
  }
  const typename ROW::elem *const token = in + (int64_t)t * p.H;
  uint64_t todo = __ballot(my_row >= 0);
  while (todo) {
    u32x4 r[R];
    int row[R], at[R];
    float a[R];
    bool in_row[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      in_row[j] = todo != 0;
      row[j] = at[j] = 0;
      a[j] = 0.0f;
      r[j] = (u32x4){0u, 0u, 0u, 0u};
      if (in_row[j]) {
        const int k = __builtin_ctzll(todo);
        todo &= todo - 1;
        row[j] = read_lane(my_row, k);
        a[j] = read_lane(my_w, k);
        in_row[j] = access::place(p, row[j], seg * kWave + lane, at[j]);
        r[j] = *(const typename access::vec *)(token + at[j]);   // inside the token's row for every lane
      }
    }
    // All reads have arrived here; left alone the compiler waits before every store, and so for the
    // store before it too (rows of 7,160 bf16, 3.6 copies: 121 us, 99 us with the one wait).
    __asm__ volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
    if constexpr (R == 8) __asm__ volatile("" : "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7]));
#pragma unroll
    for (int j = 0; j < R; ++j)
      if (in_row[j]) store_row<access>(out, p, row[j], at[j], SCALED ? ROW::scale(a[j], r[j]) : r[j]);
  }
}

// ---------------------------------------------------------------------------------------------
// Narrow rows: of fewer vectors than a wave has lanes, or of little more than a multiple of that.  One lane
// per (token, vector), tokens side by side, so that the lanes are busy however short the rows are; a lane
// reads its token's slots itself (the lanes of a token read the same words), several at a time.
// ---------------------------------------------------------------------------------------------
constexpr int kFlatThreads = 256;
constexpr int kFlatVecs = 144;   // most vectors per row that unit_of_lane divides exactly (and more than any rule asks for)

// Vectors from the row's start; the last one is moved inside the row.
template <typename ELEM>
struct NarrowRows : RaggedRows<ELEM> {
  static __device__ __forceinline__ int place(const RowParams &p, int v) {
    constexpr int P = 16 / sizeof(ELEM);
    return min(v * P, p.H - P);
  }
};

// (token, vector) of this lane, or false when past the end.  The workgroup's first unit is divided by a
// 64-bit reciprocal, the rest is a numerator n below nvec + kFlatThreads <= 400, for which the 22-bit one is
// exact: it is too large by less than nvec / 2^22 of itself, and n nvec < 2^16.
template <bool NEAR>
__device__ __forceinline__ bool unit_of_lane(const RowParams &p, int &t, int &v) {
  const int64_t first = (int64_t)block_place<NEAR>() * kFlatThreads;
  const int64_t t0 = divided(first, p.recip);
  const unsigned n = (unsigned)(first - t0 * p.nvec) + threadIdx.x;
  const unsigned dt = (n * (((1u << 22) + (unsigned)p.nvec - 1u) / (unsigned)p.nvec)) >> 22;
  t = (int)t0 + (int)dt;
  v = (int)(n - dt * (unsigned)p.nvec);
  return first + threadIdx.x < p.nunits;
}

// The rows that slots k0 .. k0 + N - 1 of token t own, -1 for a slot that owns none in [0, rows).
template <int N>
__device__ __forceinline__ void owned_rows(const RowParams &p, int t, int k0, int64_t rows, bool report, int (&row)[N]) {
  const int64_t s = (int64_t)t * p.K + k0;
  uint8_t keep[N];
  __builtin_memcpy(row, p.slot_row + s, sizeof(row));
  __builtin_memcpy(keep, p.slot_keep + s, sizeof(keep));
#pragma unroll
  for (int j = 0; j < N; ++j) {
    if (!keep[j] || row[j] < 0) {
      row[j] = -1;
    } else if (row[j] >= rows) {
      if (report) flag(p.status, HM_ERR_CAPACITY);
      row[j] = -1;
    }
  }
}

// fn(N, k0) over the K slots in pieces of eight and, WHOLE, the rest in one: a piece is a chain of trips to memory, its
// list, then its rows or weights.  Else the rest goes in pieces of four and one, which a dispatch, whose stores wait
// for nothing, prefers by 0.1 us. Combine, plan's weights, rest in pieces of four and one -> in one: 16,384 x 64, K = 7
// 8.2 -> 6.1 us, x 128, K = 3 7.5 -> 5.8, 4,096 x 256, K = 6 7.0 -> 5.5, 8,192 x 1,030, K = 6 26.1 -> 23.6; bf16
// transpose of 16,384 x 64, K = 7 7.0 -> 6.4.
template <bool WHOLE, typename FN>
__device__ __forceinline__ void for_slots(int K, FN fn) {
  int k0 = 0;
  for (; k0 + 8 <= K; k0 += 8) fn(std::integral_constant<int, 8>{}, k0);
  if constexpr (WHOLE) {
    switch (K - k0) {
      case 1: fn(std::integral_constant<int, 1>{}, k0); break;
      case 2: fn(std::integral_constant<int, 2>{}, k0); break;
      case 3: fn(std::integral_constant<int, 3>{}, k0); break;
      case 4: fn(std::integral_constant<int, 4>{}, k0); break;
      case 5: fn(std::integral_constant<int, 5>{}, k0); break;
      case 6: fn(std::integral_constant<int, 6>{}, k0); break;
      case 7: fn(std::integral_constant<int, 7>{}, k0); break;
    }
  } else {
    if (k0 + 4 <= K) {
      fn(std::integral_constant<int, 4>{}, k0);
      k0 += 4;
    }
    for (; k0 < K; ++k0) fn(std::integral_constant<int, 1>{}, k0);
  }
}

// Dispatch (SCALED = false) and transpose.  A lane reads a weight for every slot, that of row 0 for a slot
// without a row, so the transpose is launched only where there is a row 0 (rows > 0): a read
// under the slot's own condition costs 0.5 to 0.8 us (8,192 tokens, 3.6 rows of 64 bf16: 5.2 -> 6.0).
template <typename ROW, bool SCALED, bool NEAR>
__global__ __launch_bounds__(kFlatThreads) void spread_flat_kernel(RowParams p, const typename ROW::elem *__restrict__ in,
                                                                   const float *__restrict__ row_weight, int64_t rows,
                                                                   typename ROW::elem *__restrict__ out) {
  typedef NarrowRows<typename ROW::elem> access;
  int t, v;
  if (!unit_of_lane<NEAR>(p, t, v)) return;
  const int at = access::place(p, v);
  const u32x4 r = *(const typename access::vec *)(in + ((int64_t)t * p.H + at));
  for_slots<SCALED>(p.K, [&](auto n, int k0) {
    constexpr int N = decltype(n)::value;
    int row[N];
    float a[N];
    owned_rows<N>(p, t, k0, rows, v == 0, row);
#pragma unroll
    for (int j = 0; j < N; ++j) a[j] = SCALED ? row_weight[max(row[j], 0)] : 0.0f;
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (row[j] >= 0) store_row<access>(out, p, row[j], at, SCALED ? ROW::scale(a[j], r) : r);
  });
}

// Combine with the plan's weights: the sums of combine_plan_rows_kernel, in the same order.
template <bool MIX, typename ROW>
__global__ __launch_bounds__(kFlatThreads) void combine_flat_kernel(RowParams p, const typename ROW::elem *__restrict__ y,
                                                                    int64_t y_rows, const float *__restrict__ row_weight,
                                                                    typename ROW::elem *__restrict__ out) {
  typedef NarrowRows<typename ROW::elem> access;
  constexpr int E = ROW::kPerVec;
  int t, v;
  if (!unit_of_lane<false>(p, t, v)) return;
  const int at = access::place(p, v);
  float acc[E], wsum = 0.0f;
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.0f;
  for_slots<true>(p.K, [&](auto n, int k0) {
    constexpr int N = decltype(n)::value;
    int row[N];
    float a[N];
    u32x4 r[N];
    owned_rows<N>(p, t, k0, y_rows, v == 0, row);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      a[j] = 0.0f;
      r[j] = (u32x4){0u, 0u, 0u, 0u};
      if (row[j] >= 0) {
        a[j] = row_weight[row[j]];
        r[j] = load_row<access>(y, p, row[j], at);
      }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (row[j] >= 0) {
        ROW::fma_into(acc, a[j], r[j]);
        wsum = wsum + a[j];
      }
    }
  });
  if (MIX) {
    const float inv = wsum != 0.0f ? 1.0f / wsum : 0.0f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = acc[e] * inv;
  }
  store_row<access>(out, p, t, at, ROW::pack(acc));
}

template <typename ROW>
__global__ __launch_bounds__(kElemThreads) void transpose_elems_kernel(RowParams p, int32_t H,
                                                                      const typename ROW::elem *__restrict__ gout,
                                                                      const float *__restrict__ row_weight,
                                                                      int64_t weight_rows, typename ROW::elem *__restrict__ gy,
                                                                      int64_t gy_rows) {
  const int64_t i = (int64_t)blockIdx.x * kElemThreads + threadIdx.x;
  if (i >= (int64_t)p.T * H) return;
  const int t = (int)(i / H), j = (int)(i - (int64_t)t * H);
  const typename ROW::elem g = gout[i];
  for (int k = 0; k < p.K; ++k) {
    const int64_t s = (int64_t)t * p.K + k;
    const int row = p.slot_row[s];
    if (!p.slot_keep[s] || row < 0) continue;
    if (row < gy_rows && row < weight_rows) gy[(int64_t)row * H + j] = ROW::scale(row_weight[row], g);
    else if (j == 0) flag(p.status, HM_ERR_CAPACITY);
  }
}

static inline uint64_t reciprocal(int64_t d) { return d > 1 ? ~0ull / (uint64_t)d + 1 : 0; }

// Fills what the kernels need to know about rows of H elements (of 16 / per_vec bytes) written to
// `out`, and sizes the grid.  A ragged row may begin anywhere in its first line.
static inline bool grid_for_units(RowParams &p, int H, int per_vec, bool whole, const void *out, int vecs_per_lane, int block,
                                  dim3 &grid) {
  const int elem_bytes = 16 / per_vec, line = kLineBytes / elem_bytes;
  p.H = H;
  p.shift = (int)(((uintptr_t)out & (kLineBytes - 1)) / elem_bytes);
  p.nvec = (int)(((int64_t)H + (whole ? 0 : line - 1) + per_vec - 1) / per_vec);
  p.nseg = (int)(((int64_t)p.nvec + kWave * vecs_per_lane - 1) / (kWave * vecs_per_lane));
  p.nunits = (int64_t)p.T * p.nseg;
  p.recip = reciprocal(p.nseg);
  const int waves = block / kWave;
  const int64_t blocks = (p.nunits + waves - 1) / waves;
  if (blocks > 2147483647LL) return false;
  grid = dim3((unsigned)blocks);
  return true;
}

// The same for the flat kernels.
static inline bool grid_for_flat(RowParams &p, int H, int per_vec, dim3 &grid) {
  p.H = H;
  p.shift = p.nseg = 0;
  p.nvec = (H + per_vec - 1) / per_vec;
  p.nunits = (int64_t)p.T * p.nvec;
  p.recip = reciprocal(p.nvec);
  const int64_t blocks = (p.nunits + kFlatThreads - 1) / kFlatThreads;
  if (blocks > 2147483647LL) return false;
  grid = dim3((unsigned)blocks);
  return true;
}
static inline bool grid_for_elems(RowParams &p, int64_t n, dim3 &grid) {
  p.H = p.nvec = p.shift = p.nseg = 0;
  p.nunits = 0;
  p.recip = 0;
  const int64_t blocks = (n + kElemThreads - 1) / kElemThreads;
  if (blocks > 2147483647LL) return false;
  grid = dim3((unsigned)blocks);
  return true;
}

// Bytes of (unused) dynamic LDS per workgroup that leave room for `waves_per_cu` waves of
// `block`-thread workgroups on a CU; 0 = no cap.  The CU's LDS size is read from the device once.
static inline int lds_per_cu() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int v = cached[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    int bytes = 0;
    if (hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess) bytes = 0;
    v = bytes >= 65536 ? bytes : -1;
    cached[dev].store(v, std::memory_order_relaxed);
  }
  return v > 0 ? v : 0;
}
static inline unsigned lds_cap_bytes(int waves_per_cu, int block) {
  const int per_cu = lds_per_cu();
  const int blocks = waves_per_cu / (block / kWave);
  if (per_cu == 0 || blocks < 1 || waves_per_cu >= 32) return 0;
  const int bytes = (per_cu / blocks) & ~511;
  return bytes > 65536 ? 65536u : (unsigned)bytes;
}

// Rows a token is expected to own: from the caller's (or hm_plan_status's) row count if there is
// one, else from the bound hm_plan left in the struct, else unknown (0).
static inline double rows_per_token(const hm_plan_out *plan, int32_t T) {
  if (plan->expected_rows > 0 && T > 0) return (double)plan->expected_rows / (double)T;
  if (plan->max_rows_per_token > 0) return (double)plan->max_rows_per_token;
  return 0.0;
}
// The same from the row count alone, 0 if there is none: for what loses where a bound of eight stands for three rows or five.
static inline double known_rows_per_token(const hm_plan_out *plan, int32_t T) {
  return plan->expected_rows > 0 && T > 0 ? (double)plan->expected_rows / (double)T : 0.0;
}

// Waves per CU of the dispatch of whole-line rows.  A wave with seven stores for its one load wants fewer
// neighbours than one with three, as long as what it loads comes from the Infinity Cache (256 MB) and
// not from memory.  HIP events, 24 -> 12 waves: 8,192 x 2,048 at rank level (7.36 rows per token) 51.8 -> 49.3 us,
// 4,096 x 4,096 50.9 -> 48.4, 16,384 x 2,048 with 6.6 rows 86.4 -> 81.6, with 8.98 rows 123.1 -> 119.4; 8,192 x 7,168
// 164.7 -> 164.8; but 16,384 x 4,096 with 5.4 rows 145 -> 159, the DeepSeek-V3 layer (3.1 rows) 81 -> 106,
// and a token buffer of 470 MB 642 -> 651.  Only a known row count counts: the bound that hm_plan leaves is 8 for
// the layer with 5.4.
// Nor are rows of less than a segment, whose waves are short: 8,192 x 192 with 7.7 rows 5.6 -> 6.6.
static inline int dispatch_waves_per_cu(const hm_plan_out *plan, int32_t T, int32_t H) {
  const bool many = plan->expected_rows > 6 * (int64_t)T && H >= 8 * kWave;
  return many && (int64_t)T * H * 2 <= (256ll << 20) ? 12 : kCopyWavesPerCu;
}

// Whether the fp32 transpose of rows cut by WholeRows keeps dispatch's 24 waves per CU.  A wave waits once more than
// dispatch does (for the row's weight, behind its index), which more waves hide, but more waves also queue more stores.
// HIP events, graphs of ten calls, both forms in turn over two to ten pairs of buffers (one pair alone leaves gradients
// of up to 256 MB in the Infinity Cache, and capped is then up to 2 % better at many rows), capped -> uncapped in us;
// runs of one form differ by 0.5 %:
//   about one row per token: uncapped 7 to 11 % faster (8,192 x 2,048 28.4 -> 26.4, 65,536 x 2,048 202 -> 182, 65,536 x
//     7,168 680 -> 623);
//   two rows: capped (16,384 x 2,048 69.1 -> 69.9, 65,536 x 2,048 268 -> 274, 16,384 x 7,168 232 -> 243, 65,536 x 7,168
//   915 -> 977); three or four rows: uncapped (8,192 x 2,048 52.6 -> 52.1, 65,536 x 2,048 403 -> 392, 65,536 x 4,096
//   800 -> 780, 32,768 x
//     7,168 615 -> 609; 8,192 x 7,168 alone 154 -> 156);
//   seven rows: uncapped (16,384 x 2,048 194 -> 188, 32,768 x 2,048 397 -> 381, 32,768 x 4,096 806 -> 754, 65,536 x
//   2,048 844 ->
//     803, 16,384 x 7,168 726 -> 705), but capped for gradients of up to 96 MB (8,192 x 1,024 51.4 -> 53.9, 8,192 x
//     2,048 101.4 -> 104.6, 4,096 x 4,096 101.1 -> 103.7) or of more than 0.75 GB (32,768 x 7,168 1,509 -> 1,567,
//     65,536 x 7,168 2,992 -> 3,149; 65,536 x 4,096 1,661 -> 1,637).
// Rows that begin inside a line (lines = false), whose edges are written in part: capped from two rows per token on.
static inline bool transpose_capped(const hm_plan_out *plan, int32_t T, int32_t H, bool lines) {
  const double c = rows_per_token(plan, T), in = (double)T * H * 4;
  if (!lines) return c <= 0.0 || c >= 1.5;
  if (c > 6.0) return in <= (double)(96 << 20) || in > 0.75e9;
  return c <= 0.0 || (c >= 1.5 && c < 2.5);   // an unknown number of rows: capped
}

// Launch shape of the combine kernels: 16-byte vectors per lane, rows in flight per wave, and the
// cap on resident waves per CU (32 = none).  The launcher and hm_combine_launch_shape both take it from launched_shape().
struct CombineShape {
  int vecs, rows, waves_per_cu;
};
static inline CombineShape combine_shape(const hm_plan_out *plan, int32_t T, bool weights_from_plan) {
  CombineShape sh;
  if (!weights_from_plan) {
    sh.vecs = kCombineVecs;
    sh.rows = kCombineRows;
    sh.waves_per_cu = 32;
    return sh;
  }
  const double c = rows_per_token(plan, T);
  sh.waves_per_cu = 32;
  if (c <= 0.0) {   // unknown (a hop-table plan that was never synchronised): such plans have few rows per token
    sh.vecs = kCombineVecs;
    sh.rows = kCombineRows;
    return sh;
  }
  if (c < 2.0) {    // about one row per token: 1 KiB segments would be mostly prologue
    sh.vecs = kCombineVecs;
    sh.rows = kCombineRowsFew;
    return sh;
  }
  sh.vecs = 1;
  sh.rows = kCombineRowsPlan;
  int waves = 32;
  if (c > 4.0) {   // c KiB of loads per wave: keep about kCombineBytesInFlight per CU
    waves = (int)((double)kCombineBytesInFlight / (c * 1024.0));
    waves &= ~3;   // whole workgroups of four waves
    if (waves < 16) waves = 16;
    if (waves > 32) waves = 32;
  }
  sh.waves_per_cu = waves;
  return sh;
}
template <bool MIX, typename ROW, typename ACCESS>
static inline auto combine_kernel(const CombineShape &sh, bool weights_from_plan) {
  if (!weights_from_plan)
    return sh.vecs == 1 ? combine_slots_kernel<MIX, ROW, ACCESS> : combine_rows_kernel<MIX, kCombineVecs, kCombineRows, ROW, ACCESS>;
  if (sh.vecs == 1) return combine_plan_rows_kernel<MIX, 1, kCombineRowsPlan, ROW, ACCESS>;
  if (sh.rows == kCombineRowsFew) return combine_plan_rows_kernel<MIX, kCombineVecs, kCombineRowsFew, ROW, ACCESS>;
  return combine_plan_rows_kernel<MIX, kCombineVecs, kCombineRows, ROW, ACCESS>;
}

// ---------------------------------------------------------------------------------------------
// Which kernel takes the rows of a call.
// ---------------------------------------------------------------------------------------------
enum class Route {
  kWhole,    // a wave per (token, segment), WholeRows
  kRagged,   // ... RaggedRows
  kFlat,     // a lane per (token, vector)
  kElems,    // a lane per (token, element)
};

struct RowForm {
  int T, K, H, elem_bytes;
  int vecs;       // 16-byte vectors per row, the last one possibly in part
  bool vectors;   // every row of both buffers is whole, aligned vectors
  bool lines;     // ... and every row written is whole 128-byte lines
  bool apart;     // the buffers begin at different places of a line
};
static inline RowForm row_form(int T, int K, int H, int elem_bytes, const void *in, const void *out) {
  RowForm f;
  f.T = T;
  f.K = K;
  f.H = H;
  f.elem_bytes = elem_bytes;
  f.vecs = (int)(((int64_t)H * elem_bytes + 15) / 16);
  f.vectors = (int64_t)H * elem_bytes % 16 == 0 && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  f.lines = f.vectors && (int64_t)H * elem_bytes % kLineBytes == 0 && ((uintptr_t)out & (kLineBytes - 1)) == 0;
  f.apart = (((uintptr_t)in ^ (uintptr_t)out) & (kLineBytes - 1)) != 0;
  return f;
}
static inline bool in_vectors(const RowForm &f) { return f.H * (int64_t)f.elem_bytes >= 16 && f.H <= kMaxVectorH; }

// All figures below: us per call, graphs of ten calls, the kernels in turn.  Those with fresh buffers (or buffers taken
// in turn) go round enough pairs that none is still in the 256 MB Infinity Cache, as in a training step; the others use
// one pair, and the lines that they draw were measured again with fresh ones.
//
// Tokens from which a lane per vector pays where a row is whole vectors: with fewer, all waves of a wave per token are
// resident at once and a call lasts as long as one wave's chain, which is longer where a lane walks its token's K
// slots itself (512 tokens, K = 8, 64 bf16, in waves -> flat: dispatch 2.7 -> 3.0, bf16 transpose 3.6 -> 4.8; 4,096
// tokens, 7.7 rows: 4.3 -> 3.5 and 7.1 -> 5.3).  One or two slots are no such chain: combine is flat at any T there (512
// tokens, K = 1, 16 bf16: 3.2 -> 2.7).
constexpr int kFlatTokens = 4096;

// Whether the dispatch groups its workgroups by die: rows that begin inside a line, of up to 80 MB of tokens, 130 MB if
// the rows are narrow. How many rows a token has does not matter, so a plan that was never synchronised is as well off
// as one that was. Grouping helps a dispatch that is bound by its writes: tokens that the Infinity Cache (256 MB) still
// holds, as a layer's output that has just been written, or short rows, a large part of which is shared lines. HIP
// events, dispatch and a combine that reads a buffer of its own, as launched -> grouped in turn, geometric means of the
// dispatch alone over 2,200 shapes drawn (2,000 to 262,144 tokens, one to ten slots, 0.2 to ten rows per token), three
// to eight passes in turn / so many that no token is still cached:
//   128 to 1,400 bytes, up to 30 MB   +1 to +12 % / 0 to +8 %     30 to 80 MB   +2 to +13 % / 0 to +8 %     80 to 130 MB   +1 to +6 % / 0 to +9 %
//   wider rows, up to 30 MB           +2 to +6 % / -2 to +2 %     30 to 80 MB   +1 to +9 % / -2 to 0 %      more           -3 to +1 % / -5 to +2 %
// 65,536 x 136 with 3.3 rows 22.4 -> 18.4, 4.5 29.2 -> 22.0, 7.6 58.0 -> 48.8; 4,097 x 1,030 with 5.8 15.2 -> 14.3;
// 16,384 x 520 with 5.4 27.3 -> 23.6; but 8,192 x 7,161 with 3.3 108.7 -> 111.9, 75,791 x 1,039 163 -> 174. A combine
// that reads the very rows that dispatch has just written, with nothing between, finds fewer of them on its own die:
// 65,536 x 72 with one row 11.6 -> 14.1 for both.  The transpose keeps the launch order (16,384 x 2,050 with 7.7 rows
// and its combine 227.5 -> 229.7), and so do whole lines, of which neighbours share none (8,192 x 7,168 with 3.6 rows
// 159.8 -> 162.3).  Nor is there anything to group below one whole round of the dies.
static inline bool near_pays(const RowForm &f, dim3 grid) {
  const int64_t row = (int64_t)f.H * f.elem_bytes, tokens = f.T * row;
  return !f.lines && row >= 32 && tokens <= (row <= 1400 ? 130000000 : 80000000) && grid.x >= kDies * kNear;
}

// Whether the bf16 transpose of ragged rows has the reads of eight rows in flight, which hides its rounding: for up to
// eight slots that are known to be kept nearly all, and 7 MB of gradients or more.  Four -> eight, 1,300 shapes drawn,
// three to eight slots, three to eight buffers in turn, geometric means: kept nearly all, from 7 MB on 0 to +4 %
// (16,384 x 1,030 with 7.6 rows 74.7 -> 65.0 us, 8,192 x 1,030 with six 28.5 -> 26.4), below -1 to -4 % (5,114 x 363
// with 7.6 11.9 -> 12.9); 4.3 rows of six to eight slots or more 0 to +6 %, but -8 % for some (70,304 x 591 with 4.7);
// fewer rows -4 to -17 % (8,192 x 7,161 with 2.2 81.6 -> 97.3), which a bound of eight in place of a count would not
// show.  Ten rows 27.4 -> 28.1.
static inline bool eight_reads_pay(const RowForm &f, const hm_plan_out *plan) {
  const double c = known_rows_per_token(plan, f.T);
  return f.K <= 8 && c > 4.25 && c > f.K - 1 && (int64_t)f.T * f.H * f.elem_bytes >= 7000000;
}

// Dispatch (scaled = false) and transpose.
//  * Vectors, narrow: flat up to the widths at which it still gains.  65,536 tokens, 3.6 rows each, in waves -> flat:
//    dispatch of 16 bf16 13.2 -> 6.6, of 128 13.1 -> 12.1, of 256 32.8 -> 28.8 (but 32,768 tokens: 3 % slower, or 7.7
//    rows: 14 % slower); bf16 transpose of 192 32.6 -> 22.0, of 256 33.4 -> 26.9; fp32 transpose of 16 12.3 -> 5.8, of
//    64 16.9 -> 12.5, of 96 21.1 -> 19.6 (but 8,192 tokens: 5 % slower).  With K <= 2 further (K = 1: 320 bf16 16.8 ->
//    15.3). And just above 64 vectors, where waves leave most of their second segment idle: bf16 transpose (16,384
//    tokens of 576, 3.6 rows 17.7 -> 14.8; of 640 up to six rows only, with 7.7 31.5 -> 33.7; not off a line: 8,192 of
//    520 11.8 -> 12.4), dispatch for K <= 2 (K = 1: 6.7 -> 4.6; but K = 8: 12.7 -> 13.3), fp32 transpose for K = 1 (384
//    elements 8.1 -> 6.3); just above 128 for K = 1 (8,192 tokens, 1,088 bf16, dispatch 5.7 -> 4.5).
//  * Vectors, not narrow: whole lines are written by kWhole.  Rows that begin inside a line are written in line-sized
//    pieces by kRagged, which reads the token again for each row: better once that saves more in partial lines than it
//    costs, i.e. with many rows per token that are long (the extra segment for the slack of a line is a larger part of
//    short ones) and some 24 MB to write.  A weight to multiply by makes the second reading dearer, fp32 twice.  Fresh
//    buffers, packed rows 16 bytes off a line, kWhole -> kRagged, 16,384 tokens of 1,024 / 2,048 / 7,168 elements: 7.7
//    rows: dispatch 72 -> 69, 144 -> 123, 488 -> 369; bf16 transpose 79 -> 76, 158 -> 131, 533 -> 382; fp32 157 -> 124,
//    301 -> 223, 1,033 -> 839; from 36 MB on just above 64 vectors, too (584 bf16: dispatch 46.6 -> 42.9, 8,192 tokens
//    bf16 transpose 26.7 -> 23.8; but 456: 37.1 -> 39.3); 3.6 rows: dispatch 31.7 -> 32.6 (1,032: 36.4 -> 33.6), 60 ->
//    58, 202 -> 187; bf16 transpose 34.6 -> 37.2 (1,032: 37.5 -> 38.2), 64.5 -> 63.4, 210 -> 191; fp32 61 -> 68, 120 ->
//    127, 397 -> 443 (but small gradients, below 24 MB: 4,096 tokens of 512 10.1 -> 9.3, of 1,024 17.0 -> 14.3, of
//    2,048 32.5 -> 34.4; 1,024 tokens of 4,096 16.8 -> 13.8); 1.9 rows: dispatch 20.9 -> 24.2, 40.2 -> 39.8, 130 ->
//    121; bf16 transpose 22.7 -> 28.2, 42 -> 46, 131 -> 136; fp32 39 -> 50, 73 -> 95, 248 -> 319.
//  * Elements, few of them: kElems, whose lanes are all resident and have the shortest chain, for K <= 2 up to 512 Ki
//    elements (2,048 tokens, K = 1, 65 bf16, transpose: 2.7, flat 3.2, ragged 3.4), for the bf16 transpose up to 256 Ki
//    (2,048 x 33, 7.7 rows: 5.1, flat 5.6, ragged 7.6; but 16,384 x 17: 7.3, flat 6.5), for dispatch of many copies of
//    up to nine vectors up to 128 Ki (2,048 x 33: 3.9, flat 4.2; but x 100: 4.5, flat 4.0; 16 x 17: 3.5, flat 2.8).
//  * Elements, many copies of short rows: kElems, whose neighbouring lanes write neighbouring elements where vectors
//    straddle lines (65,536 tokens, 7.7 rows, fresh buffers, kElems / flat: dispatch of 17 bf16 15 / 23, of 33 27 / 33,
//    but of 65 41 / 41, of 130 84 / 61; fp32 transpose of 33 40 / 45, but of 65 69 / 65; bf16 transpose, dearer per
//    element, of 17 23 / 25, but of 33 38 / 35; and with 32,768 tokens of 17 13.7 / 12.4).
//  * Elements, narrow: flat at any number of tokens (fp32 transpose of 16 x 5, 7.8 rows: 3.0, ragged 3.9), but from
//    2,048 on for the bf16 transpose (512 x 250 5.3, ragged 5.7, but 3.6 rows 4.7 and 4.2; 2,048: 6.5 and 7.6, 5.2 and
//    5.0).  Up to 32 vectors, for fp32 with K > 2 up to 20 (65,536 tokens, 3.6 rows, ragged -> flat: 33 fp32 25 -> 16,
//    130 33 -> 39), 12 with many copies of many tokens (7.7 rows, 65 fp32: 57 -> 65, but 8,192 tokens 9.2 -> 8.6), for
//    K = 1 up to 76, as far as the ragged kernel's slack of a line fills a second segment badly (65,536 x 250 fp32: 55
//    -> 28); else ragged (7.3 copies of 301 bf16: 113, flat 116).
static inline Route spread_route(const RowForm &f, const hm_plan_out *plan, bool scaled) {
  if (!in_vectors(f)) return Route::kElems;
  const bool wide = f.elem_bytes == 4, scaled_bf16 = scaled && !wide;
  const int64_t elems = (int64_t)f.T * f.H;
  const double rows = rows_per_token(plan, f.T), bytes = (double)elems * f.elem_bytes;
  if (f.vectors) {
    const bool enough = rows > 6.0   ? f.vecs > (bytes * rows >= 36e6 ? kWave : 120)
                        : rows > 2.5 ? (wide ? bytes < 24e6 && f.vecs >= 2 * kWave : f.vecs >= (scaled ? 4 * kWave : 2 * kWave + 1))
                                     : rows > 1.5 && !scaled && f.vecs >= 4 * kWave;
    const bool ragged = !f.lines && enough && bytes * rows >= 24e6;
    const int many = f.T >= 65536 && rows <= 6.0 ? 32 : 16;
    const int narrow = f.K == 1 ? 48 : f.K == 2 ? (wide ? 24 : 48) : wide ? 16 : scaled ? 32 : many;
    const int above = f.K == 1 ? (wide ? 96 : 88) : f.K == 2 ? (wide ? 0 : 80) : scaled_bf16 && f.lines ? (rows > 6.0 ? 72 : 80) : 0;
    const bool few_lanes =   // in the last segment
        (f.vecs > kWave && f.vecs <= above) || (f.K == 1 && f.vecs > 2 * kWave && f.vecs <= kFlatVecs);
    if (f.T >= kFlatTokens && (f.vecs <= narrow || (few_lanes && !ragged))) return Route::kFlat;
    return ragged ? Route::kRagged : Route::kWhole;
  }
  const bool many_copies = plan->expected_rows > 6 * (int64_t)f.T;
  const bool few = f.K <= 2       ? elems <= 512 * 1024
                   : scaled_bf16 ? elems <= 256 * 1024
                                 : !wide && many_copies && elems <= 128 * 1024 && f.T >= 256 && f.vecs <= 9;
  if (few || (many_copies && f.T >= (scaled_bf16 ? 65536 : 32768) && f.vecs <= (wide ? 9 : scaled ? 3 : 5))) return Route::kElems;
  const int narrow = f.K == 1 ? 76 : wide && f.K > 2 ? (many_copies && f.T >= 32768 ? 12 : 20) : 32;
  return f.vecs <= narrow && (!scaled_bf16 || f.T >= 2048) ? Route::kFlat : Route::kRagged;
}

// With the caller's weights: segments of 1 KiB (combine_slots_kernel, under combine_shape's cap) or of 4 KiB
// (combine_rows_kernel) for tokens known to have two rows or more.  Rows of one short segment always: the lanes of a
// long one would be idle.  Longer rows where the waves of short segments still run all at once (16 per CU), as each has
// less to wait for, and where not even those of long ones do, if there are bytes enough to hide that every segment
// finds the token's rows again, three rows or so for each, and few idle lanes in the last segment.  HIP events, buffers
// in turn, 4 KiB -> 1 KiB, us: 8,192 x 256 bf16 with 7 rows 15.0 -> 10.2, 16,384 x 512 with 4 22.6 -> 16.6; 1,024 x
// 1,030 7.5 -> 6.2, but 4,096 x 1,030 14.8 -> 16.6, 4,096 x 640 10.4 -> 11.0, 4,096 x 1,792 with 5 8 % slower; 8,192 x
// 7,160 158.8 -> 153.6, 3,072 x 2,304 up to 7 % faster, 32,768 x 1,920 8 %, but 16,384 x 1,030 50.7 -> 57.2 and x 4,097
// 4 % slower.  Of two rows: 32,768 x 1,664 9 % slower, 2,048 x 7,168 4 %.  Only a known row count counts: tokens of one
// row or so under a bound of eight take 49 -> 81 us (8,192 x 7,168 bf16, 1.2 rows), 18 -> 25 (x 2,048), 62 -> 96
// (32,768 x 2,048, 1.6 rows), which is more than the 3 to 12 % that those of many rows would gain.
static inline bool short_segments(const RowForm &f, const hm_plan_out *plan) {
  const double rows = known_rows_per_token(plan, f.T);
  if (rows < 2.0) return false;
  if (f.vecs <= kWave) return true;
  constexpr int64_t kAtOnce = 4096;
  const int64_t segments = (f.vecs + kWave - 1) / kWave, of_long = (f.vecs + kCombineVecs * kWave - 1) / (kCombineVecs * kWave);
  if (f.T * segments <= kAtOnce) return true;
  return f.T * of_long > kAtOnce && (int64_t)f.T * f.vecs * 16 >= 14000000 && rows >= 2.5 &&
         10 * (int64_t)f.vecs >= 9 * kWave * segments;
}
static inline CombineShape launched_shape(const RowForm &f, const hm_plan_out *plan, bool weights_from_plan) {
  return combine_shape(plan, f.T, weights_from_plan || short_segments(f, plan));
}

// Combine; vecs_per_lane is that of the wave kernels' launch shape.
//  * With the caller's weights there is no flat kernel.  Elements: kElems where K slots of H elements are less work
//    than a wave's merging of the slots (65,536 tokens, fresh buffers, kElems / ragged: K = 1, 99 bf16 23 / 38, 161 46
//    / 40; K = 2, 65 33 / 50, 99 58 / 51; K = 8, 3.6 rows, 17 53 / 70; K = 4, fp32, 17 27 / 39, 33 55 / 40; K = 1,
//    fp32, 99 32 / 30) or there are few of them (1,024 tokens, K = 1, 513: 3.5 / 4.0), as long as its chain over K
//    slots squared is hidden (8,192 tokens, K = 8, 17 elements: 14.3 / 11.1).
//  * With the plan's weights.  Vectors: flat where narrow (65,536 tokens, 3.6 rows, in waves -> flat: 64 bf16 27.6 ->
//    9.4, 320 35.1 -> 32.2, 384 38.3 -> 37.7; 64 fp32 27.7 -> 14.5, 100 31.3 -> 22.7; K = 1 further, 16,384 x 456 bf16
//    11.0 -> 8.6), and where segments of one vector per lane would leave the last one mostly idle (16,384 tokens, 576
//    bf16: 18.6 -> 16.1, 1,088 28.8 -> 27.3, 320 fp32 18.5 -> 16.6); segments of four only for K = 1 (65 to 88 bf16
//    vectors 4 to 30 %, 320 fp32 16,384 tokens 10.2 -> 9.7, 65,536 32.9 -> 29.1) or few tokens of bf16 (1,024 x 1,000,
//    K = 1: 3.4 -> 3.0; 8,192 x 576, K = 2: equal, 1,152 20 % slower).  Elements: flat where waves would have a quarter
//    of their lanes idle or more (65,536 tokens, 3.6 rows, 301 bf16: ragged 40, flat 39, kElems 344) or, for K = 1,
//    three of four vectors of a lane (65,536 x 451: ragged 37, flat 28), kElems for K <= 2 and few elements (2,048
//    tokens, K = 1, 65 bf16: 2.6, flat 3.1).
//  * In waves: kWhole for whole lines and where the slack of a line would cost kRagged one more segment, of few or long
//    ones (4,096 tokens, K = 1, 2,048 bf16 16 bytes off a line, the caller's weights: 6.4 whole, 9.4 ragged) or with
//    reads off a line that kWhole would do in lines (8,192 x 4,096, 7.7 rows, only out off a line: 97 and 101); else
//    kRagged (16,384 x 7,168, 3.6 rows, both 16 bytes off: bf16 173 whole, 163 ragged; fp32 354 and 326).
static inline Route combine_route(const RowForm &f, bool from_plan, int vecs_per_lane) {
  if (!in_vectors(f)) return Route::kElems;
  const bool wide = f.elem_bytes == 4, many = f.T >= kFlatTokens || f.K <= 2;
  const int64_t elems = (int64_t)f.T * f.H;
  const int slack = kLineBytes / 16 - 1, segment = kWave * vecs_per_lane;
  const bool extra = (f.vecs + slack + segment - 1) / segment > (f.vecs + segment - 1) / segment;   // segment for the slack
  const bool dear = extra && (vecs_per_lane > 1 || f.vecs < 8 * kWave || f.apart);
  const Route waves = f.vectors && (f.lines || f.vecs <= kWave || dear) ? Route::kWhole : Route::kRagged;
  if (!from_plan) {
    if (f.vectors) return waves;
    const bool light = (int64_t)f.H * f.K <= (wide ? 90 : 150) || elems <= 512 * 1024 / (f.K * f.K);
    return light && (f.K <= 2 || f.T >= 2048 * f.K) ? Route::kElems : waves;
  }
  if (f.vectors) {
    const bool few_lanes = (f.vecs > kWave && f.vecs <= 88) || (f.vecs > 2 * kWave && f.vecs <= kFlatVecs);   // in the last segment
    const bool above = vecs_per_lane == 1 ? few_lanes && f.T >= kFlatTokens
                       : f.vecs > kWave && f.vecs <= (!wide && f.K <= 2 && f.T <= 1024 ? kFlatVecs : f.K == 1 ? 88 : 0);
    const bool flat = f.vecs <= (f.K == 1 ? kWave : wide ? 32 : 48) || above;
    return many && flat ? Route::kFlat : waves;
  }
  if (f.K <= 2 && elems <= 512 * 1024) return Route::kElems;
  const int in_waves = f.vecs + slack, lanes = (in_waves + kWave - 1) / kWave * kWave;
  const bool idle = 4 * in_waves <= 3 * lanes || (f.K == 1 && f.vecs <= kWave);
  return many && f.vecs <= kFlatVecs && idle ? Route::kFlat : waves;
}

}  // namespace hm

static hm_status check_rows_args(int32_t T, int32_t K, int32_t H, const hm_plan_out *plan, bool need_keep) {
  if (!plan) return HM_ERR_NULL;
  if (!plan->slot_row || !plan->status || (need_keep && !plan->slot_keep)) return HM_ERR_NULL;
  hm_status st = hm_check_tk(T, K);
  if (st != HM_OK) return st;
  if (H < 1) return HM_ERR_SHAPE;
  return HM_OK;
}

extern "C" hm_status hm_dispatch_pack(const void *x_bf16, int32_t T, int32_t K, int32_t H, const hm_plan_out *plan,
                                      void *packed_bf16, int64_t packed_rows, void *hip_stream) {
  HM_ENTRY_SCOPE;
  using namespace hm;
  hm_status st = check_rows_args(T, K, H, plan, true);
  if (st != HM_OK) return st;
  if (packed_rows < 0) return HM_ERR_SHAPE;
  if (T == 0) return HM_OK;
  if (!x_bf16 || (!packed_bf16 && packed_rows > 0)) return HM_ERR_NULL;
  hipStream_t stream = (hipStream_t)hip_stream;
  RowParams p;
  p.T = T;
  p.K = K;
  p.slot_row = plan->slot_row;
  p.slot_keep = plan->slot_keep;
  p.status = plan->status;
  dim3 grid;
  const uint16_t *x = (const uint16_t *)x_bf16;
  uint16_t *packed = (uint16_t *)packed_bf16;
  const RowForm form = row_form(T, K, H, 2, x_bf16, packed_bf16);
  const Route route = spread_route(form, plan, false);
  if (route == Route::kFlat) {
    if (!grid_for_flat(p, H, 8, grid)) return HM_ERR_SHAPE;
    const bool near = near_pays(form, grid);
    hipLaunchKernelGGL((near ? spread_flat_kernel<RowBf16, false, true> : spread_flat_kernel<RowBf16, false, false>), grid,
                       dim3(kFlatThreads), 0, stream, p, x, nullptr, packed_rows, packed);
  } else if (route != Route::kElems) {
    const bool whole = route == Route::kWhole;
    if (!grid_for_units(p, H, 8, whole, packed_bf16, 1, kCopyThreads, grid)) return HM_ERR_SHAPE;
    const bool near = near_pays(form, grid);
    const unsigned lds = lds_cap_bytes(form.lines ? dispatch_waves_per_cu(plan, T, H) : kCopyWavesPerCu, kCopyThreads);
    if (whole)
      hipLaunchKernelGGL((near ? dispatch_rows_kernel<true> : dispatch_rows_kernel<false>), grid, dim3(kCopyThreads), lds, stream, p, x,
                         packed, packed_rows);
    else
      hipLaunchKernelGGL((near ? spread_ragged_kernel<RowBf16, false, 4, true> : spread_ragged_kernel<RowBf16, false, 4, false>),
                         grid, dim3(kCopyThreads), lds, stream, p, x, nullptr, packed_rows, packed);
  } else {
    if (!grid_for_elems(p, (int64_t)T * H, grid)) return HM_ERR_SHAPE;
    hipLaunchKernelGGL(dispatch_elems_kernel, grid, dim3(kElemThreads), 0, stream, p, H, x, packed, packed_rows);
  }
  return hm_launch_status();
}

template <bool MIX, typename ROW>
static hm_status launch_combine(const void *y, int64_t y_rows, const float *topk_weights, int32_t T, int32_t K,
                                int32_t H, const hm_plan_out *plan, void *out, void *hip_stream) {
  using namespace hm;
  typedef typename ROW::elem elem;
  const bool from_plan = topk_weights == nullptr;   // merged weights and first-slot marks of the plan
  hm_status st = check_rows_args(T, K, H, plan, from_plan);
  if (st != HM_OK) return st;
  if (from_plan && !plan->row_weight) return HM_ERR_NULL;
  if (y_rows < 0 || (from_plan && plan->row_capacity < 0)) return HM_ERR_SHAPE;
  if (T == 0) return HM_OK;
  if (!out || (!y && y_rows > 0)) return HM_ERR_NULL;
  hipStream_t stream = (hipStream_t)hip_stream;
  RowParams p;
  p.T = T;
  p.K = K;
  p.slot_row = plan->slot_row;
  p.slot_keep = plan->slot_keep;
  p.status = plan->status;
  dim3 grid;
  // rows the plan's weight array does not cover are treated like rows beyond y
  const int64_t rows = from_plan && plan->row_capacity < y_rows ? plan->row_capacity : y_rows;
  const RowForm form = row_form(T, K, H, sizeof(elem), y, out);
  const CombineShape sh = launched_shape(form, plan, from_plan);
  const Route route = combine_route(form, from_plan, sh.vecs);
  if (route == Route::kFlat) {
    if (!grid_for_flat(p, H, ROW::kPerVec, grid)) return HM_ERR_SHAPE;
    hipLaunchKernelGGL((combine_flat_kernel<MIX, ROW>), grid, dim3(kFlatThreads), 0, stream, p, (const elem *)y, rows,
                       plan->row_weight, (elem *)out);
  } else if (route != Route::kElems) {
    const bool whole = route == Route::kWhole;
    if (!grid_for_units(p, H, ROW::kPerVec, whole, out, sh.vecs, kCombineThreads, grid)) return HM_ERR_SHAPE;
    const float *weights = from_plan ? plan->row_weight : topk_weights;
    const unsigned lds = sh.vecs == 1 ? lds_cap_bytes(sh.waves_per_cu, kCombineThreads) : 0u;
    const auto kernel = whole ? combine_kernel<MIX, ROW, WholeRows<elem>>(sh, from_plan)
                              : combine_kernel<MIX, ROW, RaggedRows<elem>>(sh, from_plan);
    hipLaunchKernelGGL(kernel, grid, dim3(kCombineThreads), lds, stream, p, (const elem *)y, rows, weights, (elem *)out);
  } else {
    if (!grid_for_elems(p, (int64_t)T * H, grid)) return HM_ERR_SHAPE;
    // the element-wise kernel finds the first slot of each row itself and takes the row's merged
    // weight from the plan when the caller passed none
    hipLaunchKernelGGL((combine_elems_kernel<MIX, ROW>), grid, dim3(kElemThreads), 0, stream, p, H, (const elem *)y,
                       rows, topk_weights,
                       from_plan ? plan->row_weight : nullptr, (elem *)out);
  }
  return hm_launch_status();
}

extern "C" hm_status hm_combine_launch_shape(int32_t T, int32_t K, int32_t H, const hm_plan_out *plan,
                                             int32_t weights_from_plan, int32_t *vectors_per_lane,
                                             int32_t *rows_in_flight, int32_t *waves_per_cu) {
  HM_ENTRY_SCOPE;
  hm_status st = check_rows_args(T, K, H, plan, false);
  if (st != HM_OK) return st;
  const hm::RowForm rows = hm::row_form(T, K, H, 2, nullptr, nullptr);   // of bf16, aligned
  const hm::CombineShape sh = hm::launched_shape(rows, plan, weights_from_plan != 0);
  if (vectors_per_lane) *vectors_per_lane = sh.vecs;
  if (rows_in_flight) *rows_in_flight = sh.rows;
  if (waves_per_cu) *waves_per_cu = sh.waves_per_cu;
  return HM_OK;
}

extern "C" hm_status hm_combine(const void *y_bf16, int64_t y_rows, const float *topk_weights, int32_t T, int32_t K,
                                int32_t H, const hm_plan_out *plan, void *out_bf16, void *hip_stream) {
  HM_ENTRY_SCOPE;
  return launch_combine<false, hm::RowBf16>(y_bf16, y_rows, topk_weights, T, K, H, plan, out_bf16, hip_stream);
}

extern "C" hm_status hm_combine_f32(const float *y, int64_t y_rows, const float *topk_weights, int32_t T, int32_t K,
                                    int32_t H, const hm_plan_out *plan, float *out, void *hip_stream) {
  HM_ENTRY_SCOPE;
  return launch_combine<false, hm::RowF32>(y, y_rows, topk_weights, T, K, H, plan, out, hip_stream);
}

extern "C" hm_status hm_combine_mix(const void *y_bf16, int64_t y_rows, const float *row_weights, int32_t T, int32_t K,
                                    int32_t H, const hm_plan_out *plan, void *out_bf16, void *hip_stream) {
  HM_ENTRY_SCOPE;
  return launch_combine<true, hm::RowBf16>(y_bf16, y_rows, row_weights, T, K, H, plan, out_bf16, hip_stream);
}

template <typename ROW>
static hm_status launch_transpose(const void *gout, int32_t T, int32_t K, int32_t H, const hm_plan_out *plan, void *gy,
                                  int64_t gy_rows, void *hip_stream) {
  using namespace hm;
  typedef typename ROW::elem elem;
  hm_status st = check_rows_args(T, K, H, plan, true);
  if (st != HM_OK) return st;
  if (!plan->row_weight) return HM_ERR_NULL;
  if (gy_rows < 0 || plan->row_capacity < 0) return HM_ERR_SHAPE;
  if (T == 0) return HM_OK;
  if (!gout || (!gy && gy_rows > 0)) return HM_ERR_NULL;
  hipStream_t stream = (hipStream_t)hip_stream;
  RowParams p;
  p.T = T;
  p.K = K;
  p.slot_row = plan->slot_row;
  p.slot_keep = plan->slot_keep;
  p.status = plan->status;
  dim3 grid;
  const int64_t rows = plan->row_capacity < gy_rows ? plan->row_capacity : gy_rows;
  const RowForm form = row_form(T, K, H, sizeof(elem), gout, gy);
  Route route = spread_route(form, plan, true);
  if (route == Route::kFlat && rows == 0) route = Route::kElems;   // the flat kernel reads the weight of row 0
  if (route == Route::kFlat) {
    if (!grid_for_flat(p, H, ROW::kPerVec, grid)) return HM_ERR_SHAPE;
    hipLaunchKernelGGL((spread_flat_kernel<ROW, true, false>), grid, dim3(kFlatThreads), 0, stream, p, (const elem *)gout,
                       plan->row_weight, rows, (elem *)gy);
  } else if (route != Route::kElems) {
    const bool whole = route == Route::kWhole;
    if (!grid_for_units(p, H, ROW::kPerVec, whole, gy, 1, kCopyThreads, grid)) return HM_ERR_SHAPE;
    const bool capped = ROW::kPerVec == 4 && (!whole || transpose_capped(plan, T, H, form.lines));
    const unsigned lds = capped ? lds_cap_bytes(kCopyWavesPerCu, kCopyThreads) : 0u;
    if (whole) {
      const bool divide = ROW::kPerVec == 8 && (double)T * H * 2 * rows_per_token(plan, T) > 2e9;   // bytes written
      hipLaunchKernelGGL((divide ? transpose_rows_kernel<ROW, ROW::kPerVec == 8> : transpose_rows_kernel<ROW, false>), grid,
                         dim3(kCopyThreads), lds, stream, p, (const elem *)gout, plan->row_weight, plan->row_capacity,
                         (elem *)gy, gy_rows);
    } else {
      constexpr bool bf16 = std::is_same_v<ROW, RowBf16>;
      const bool eight = bf16 && eight_reads_pay(form, plan);
      hipLaunchKernelGGL((eight ? spread_ragged_kernel<ROW, true, bf16 ? 8 : 4, false> : spread_ragged_kernel<ROW, true, 4, false>), grid,
                         dim3(kCopyThreads), lds, stream, p, (const elem *)gout, plan->row_weight, rows, (elem *)gy);
    }
  } else {
    if (!grid_for_elems(p, (int64_t)T * H, grid)) return HM_ERR_SHAPE;
    hipLaunchKernelGGL((transpose_elems_kernel<ROW>), grid, dim3(kElemThreads), 0, stream, p, H, (const elem *)gout,
                       plan->row_weight, plan->row_capacity, (elem *)gy, gy_rows);
  }
  return hm_launch_status();
}

extern "C" hm_status hm_combine_transpose(const float *gout, int32_t T, int32_t K, int32_t H, const hm_plan_out *plan,
                                          float *gy, int64_t gy_rows, void *hip_stream) {
  HM_ENTRY_SCOPE;
  return launch_transpose<hm::RowF32>(gout, T, K, H, plan, gy, gy_rows, hip_stream);
}

extern "C" hm_status hm_combine_transpose_bf16(const void *gout_bf16, int32_t T, int32_t K, int32_t H,
                                               const hm_plan_out *plan, void *gy_bf16, int64_t gy_rows, void *hip_stream) {
  HM_ENTRY_SCOPE;
  return launch_transpose<hm::RowBf16>(gout_bf16, T, K, H, plan, gy_bf16, gy_rows, hip_stream);
}
