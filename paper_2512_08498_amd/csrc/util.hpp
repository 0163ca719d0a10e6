// Wavefront (64 lanes) and workgroup scan / reduction helpers.
#pragma once

#include "common.hpp"

namespace gsr {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / kWave; }

// Inclusive prefix sum over the wave.
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T x) {
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T y = __shfl_up(x, d, kWave);
    if (lane >= d) x += y;
  }
  return x;
}

// Exclusive prefix sum over a workgroup of NT threads; `total` gets the sum.
// `lds` must hold NT / 64 elements.  Contains two barriers.
template <int NT, typename T>
__device__ __forceinline__ T block_excl_scan(T x, T *lds, T &total) {
  constexpr int NW = NT / kWave;
  const T incl = wave_incl_scan(x);
  if (lane_id() == kWave - 1) lds[wave_id()] = incl;
  __syncthreads();
  T before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const T s = lds[w];
    if (w < wave_id()) before += s;
    sum += s;
  }
  __syncthreads();
  total = sum;
  return before + incl - x;
}

// Four floats at any float's address (one load or store all the same).
struct __attribute__((packed, aligned(4))) Loose4 {
  float x, y, z, w;
};

template <typename T>
__device__ __forceinline__ T wave_reduce_or(T x) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) x |= __shfl_xor(x, d, kWave);
  return x;
}

template <typename T>
__device__ __forceinline__ T wave_reduce_and(T x) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) x &= __shfl_xor(x, d, kWave);
  return x;
}

template <typename T>
__device__ __forceinline__ T wave_reduce_max(T x) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T y = __shfl_xor(x, d, kWave);
    x = x > y ? x : y;
  }
  return x;
}

// Swap-and-add of two values a, b over the wave's halves: lanes 0..31 get
// a[l] + a[l + 32], lanes 32..63 get b[l - 32] + b[l].
__device__ __forceinline__ float fold32(float a, float b) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// Swap-and-add of two fold32 results x (values A | B) and y (C | D): lanes
// 0..15 get A, 16..31 get C, 32..47 get B, 48..63 get D, each added up over
// the rows of 16 lanes.
__device__ __forceinline__ float fold16(float x, float y) {
  const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// keep + (send of the DPP partner CTRL), in float.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float keep, float send) {
  return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), CTRL, 0xF, 0xF, false));
}

// Exchange-and-add of two values between DPP partners that differ in lane
// bit `hi`: the lane with the bit clear keeps a, the other keeps b, and each
// adds its partner's copy of the value it keeps.
template <int CTRL>
__device__ __forceinline__ float pack_add(float a, float b, bool hi) {
  return dpp_add<CTRL>(hi ? b : a, hi ? a : b);
}

// Wave sums of nine values, with the values packed as the reduction goes: the
// 32- and 16-lane swaps fold two values into one register with one add each
// (9 -> 5 -> 3), rotate 8 and the half-row mirror keep one value of a pair per
// lane (3 -> 2 -> 1), and the quad permutes complete the sums: 25
// instructions (33 when the pairwise steps came first, at two selects a pair).
// On return sum9_value says whose sum a lane holds.  Fixed order
// (deterministic); every lane must be active.
__device__ __forceinline__ float wave_sum9_packed(const float (&v)[9]) {
  const int l = lane_id();
  const bool b2 = (l >> 2) & 1, b3 = (l >> 3) & 1;
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kRor8 = 0x128, kHalfMirror = 0x141;
  const float a = fold32(v[0], v[1]), b = fold32(v[2], v[3]);
  const float c = fold32(v[4], v[5]), d = fold32(v[6], v[7]), e = fold32(v[8], v[8]);
  // rows of 16 lanes: x = (v0, v2, v1, v3), y = (v4, v6, v5, v7), z = v8
  const float x = fold16(a, b), y = fold16(c, d), z = fold16(e, e);
  const float t = pack_add<kRor8>(x, y, b3);       // x in lanes 0..7 of a row, y in 8..15
  const float r = pack_add<kHalfMirror>(t, dpp_add<kRor8>(z, z), b2);  // z in lanes with bit 2
  const float s = dpp_add<kXor1>(r, r);
  return dpp_add<kXor2>(s, s);
}

// The value whose sum this lane is to write after wave_sum9_packed, or -1: each
// is in the four lanes of a quad, of which the first writes it.
__device__ __forceinline__ int sum9_value(int lane) {
  if (lane == 4) return 8;
  return (lane & 7) ? -1 : (lane >> 5) | ((lane >> 3) & 2) | ((lane >> 1) & 4);
}

// Lanes below this one in the wave.
__device__ __forceinline__ uint64_t lanemask_lt() { return (uint64_t(1) << lane_id()) - 1u; }

// Atomic increment of *p for every lane with `pred`, issued once per wave:
// each such lane gets a distinct old value (in lane order within the wave).
// Must be reached by all lanes of the wave.
__device__ __forceinline__ uint32_t wave_atomic_inc(uint32_t *p, bool pred) {
  const uint64_t m = __ballot(pred);
  if (m == 0) return 0u;
  const int leader = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0u;
  if (lane_id() == leader) base = atomicAdd(p, (uint32_t)__popcll(m));
  base = __shfl(base, leader, kWave);
  return base + (uint32_t)__popcll(m & lanemask_lt());
}

// Tile visited by workgroup `bid` of a grid of `grid` workgroups over `total`
// tiles.  Consecutive workgroups are dispatched round-robin over the 8 XCDs;
// this mapping gives each XCD one contiguous run of tiles so neighbouring
// tiles, which share most of their Gaussians, hit the same L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t bid, uint32_t grid) {
  const uint32_t per_xcd = grid / 8u;  // grid is a multiple of 8
  return (bid % 8u) * per_xcd + bid / 8u;
}

__device__ __forceinline__ int view_of_tile(const ViewInfo *__restrict__ views, int n_views, uint32_t tile) {
  int v = 0;
  while (v + 1 < n_views && views[v + 1].tile_base <= tile) ++v;
  return v;
}

// The same for a tile that is the same in all lanes of the wave: one ballot
// per 64 views instead of a chain of dependent loads (20 of them on average
// over 40 views).  Every lane of the wave must call it.
__device__ __forceinline__ int wave_view_of_tile(const ViewInfo *__restrict__ views, int n_views, uint32_t tile) {
  int v = -1;
  for (int b = 0; b < n_views; b += kWave) {
    const int i = b + lane_id();
    v += __popcll(__ballot(i < n_views && views[i].tile_base <= tile));
  }
  return v;
}

}  // namespace gsr
