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
