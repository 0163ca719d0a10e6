// Tile geometry shared by the forward and backward compositing kernels.
//
// Pixels are walked in blocks of 8 x 8, one per lane, mostly a wave per block
// (the backward's short 16 px lists: four blocks per wave, so the per-record
// wave reduction is paid once for all four).  A lane tests a record against
// the block or tile, ballots keep the records that can composite there, and
// the wave reads those from LDS as broadcasts.  A workgroup takes one work
// item, or (a tuning option) persistent workgroups take items from a work
// queue; longest lists come first.
//
// Per pixel and Gaussian, with the record's payload (see common.hpp):
//   dx = (px - i0) - offx,  dy = (py - j0) - offy
//   u  = dx + qb dy
//   q  = qa u^2 + qc dy^2            (= log2 of the Gaussian falloff)
//   alpha = min(0.99, opacity * 2^q)
// which is the conic quadratic form -(a dx^2 + 2 b dx dy + c dy^2)/2 written
// as a sum of squares, free of the cancellation the expanded form suffers
// for elongated footprints.
//
// The tile lists hold every tile of a record's binning rectangle, but the
// alpha >= 1/255 ellipse of an elongated or tilted footprint misses many of
// them, and most of a tile's blocks.  The test (tile_reaches) is
// conservative, so the composited sequence of every pixel is unchanged.
#pragma once

#include <algorithm>
#include <atomic>

#include "common.hpp"
#include "util.hpp"

namespace gsr {

// Whether the record (box, p1, p2 of its payload) can reach alpha >= 1/255 at
// a pixel of the tile whose pixels span [x0, x0 + ts - 1] x [y0, y0 + ts - 1].
// With A = -qa, C = -qc, k = qb the falloff is f = A (dx + k dy)^2 + C dy^2
// (alpha = opacity 2^-f), convex, and a pixel composites only if
// f <= log2(255 opacity).  Its exact minimum over the rectangle tile ∩ box
// (continuous, so it bounds every pixel centre in it) is 0 when the
// rectangle holds the centre, else the least of the four edge minima: at
// fixed dy the minimiser is dx = -k dy, at fixed dx it is
// dy = -A k dx / (A k^2 + C), each clamped to the edge.  The record is
// dropped only if that minimum exceeds the threshold by a margin covering the
// rounding of this evaluation and of the per-pixel one (a relative 2^-18 of
// the largest value f takes on the rectangle, plus 1/16 for the hardware
// exp2 and log2); NaN keeps it.
__device__ __forceinline__ bool tile_reaches(const float4 box, const float4 p1, const float4 p2, float x0, float y0,
                                             float ts) {
  const float X0 = fmaxf(x0, box.x), X1 = fminf(x0 + (ts - 1.0f), box.y);
  const float Y0 = fmaxf(y0, box.z), Y1 = fminf(y0 + (ts - 1.0f), box.w);
  if (X0 > X1 || Y0 > Y1) return false;
  const float dx0 = (X0 - box.x) - p1.x, dx1 = (X1 - box.x) - p1.x;
  const float dy0 = (Y0 - box.z) - p1.y, dy1 = (Y1 - box.z) - p1.y;
  const float A = -p1.z, k = p1.w, C = -p2.x;
  auto f = [&](float dx, float dy) {
    const float u = fmaf(k, dy, dx);
    return fmaf(A, u * u, C * (dy * dy));
  };
  auto clampf = [](float v, float lo, float hi) { return fminf(fmaxf(v, lo), hi); };
  float fmin = 0.0f;
  if (!(dx0 <= 0.0f && dx1 >= 0.0f && dy0 <= 0.0f && dy1 >= 0.0f)) {
    const float r = (A * k) / fmaf(A * k, k, C);
    const float e0 = f(clampf(-k * dy0, dx0, dx1), dy0), e1 = f(clampf(-k * dy1, dx0, dx1), dy1);
    const float e2 = f(dx0, clampf(-r * dx0, dy0, dy1)), e3 = f(dx1, clampf(-r * dx1, dy0, dy1));
    fmin = fminf(fminf(e0, e1), fminf(e2, e3));
  }
  const float mx = fmaxf(fabsf(dx0), fabsf(dx1)), my = fmaxf(fabsf(dy0), fabsf(dy1));
  const float um = fmaf(fabsf(k), my, mx);
  const float big = fmaf(A, um * um, C * (my * my));
  const float thr = __builtin_amdgcn_logf(p2.y) + 0x1.ffa37cp+2f;  // log2(opacity) + log2(255)
  return !(fmin > thr + (0.0625f + 0x1p-18f * big));
}

// Persistent compositing launches: as many workgroups as the chip holds at
// once, each walking work items (tiles, or groups of tiles, in the
// longest-first order) until none is left; taking an item never waits for
// another workgroup, so the balance adapts at run time to the actual cost of
// each list.  Item i belongs to lane i % 8 of the queue, and workgroup b
// serves lane b % 8: its first item is b itself, later ones come from that
// lane's counter, one atomic add per item (lane-local index gridDim.x / 8 +
// count).  The grid is a multiple of eight, so every lane has workgroups and
// every item is taken exactly once, however the workgroups are placed.  The
// chip dispatches workgroups to its eight XCDs round-robin, so each counter
// (on a 128-byte line of its own) is used from one XCD: the eight are served
// in parallel, where a single counter for all workgroups serialised the
// atomics and doubled the compositing time.  The add for the next item is
// issued when the current one starts (a wave's memory returns complete in
// order, so it is still waited for at the walk's first load, which overlaps
// most of its latency).  A workgroup stops at its first item past the end;
// the claim it still has in flight then lies past the end too (a lane's
// items grow with its count), so no item is lost.  The counters start at
// zero: the forward's first kernel zeroes both queues, and the pair
// reduction that follows every compositing backward zeroes the backward's
// again.
// Without persistence (P = false) the grid has one workgroup per item and
// next() ends the walk after the first; the kernels are instantiated for
// both, so the grid schedule carries no queue state.
template <bool P>
struct ItemQueue {
  uint32_t *ctr;   // the lane's counter
  uint32_t claim;  // thread 0: lane-local count claimed for the next item

  __device__ __forceinline__ explicit ItemQueue(uint32_t *queue)
      : ctr(queue + (blockIdx.x & (kQueueLanes - 1u)) * kQueueStride), claim(0u) {
    if (P && threadIdx.x == 0) claim = atomicAdd(ctr, 1u);
  }

  // Next item of the calling workgroup (uniform); every thread must call it,
  // after its last access to the LDS of the current item.
  __device__ __forceinline__ uint32_t next(uint32_t *slot) {
    if (!P) return 0xFFFFFFFFu;
    if (threadIdx.x == 0) *slot = claim;
    __syncthreads();
    const uint32_t k = *slot;
    __syncthreads();
    if (threadIdx.x == 0) claim = atomicAdd(ctr, 1u);
    return (gridDim.x / kQueueLanes + k) * kQueueLanes + (blockIdx.x & (kQueueLanes - 1u));
  }
};

// Workgroups of a persistent launch: the current device's compute units times
// the workgroups of Kernel (of `threads` threads) that one holds at once, a
// multiple of the queue's lanes.  Asked of the runtime once per kernel and
// device; the kernel is a template argument, as kernels of one signature hold
// from two to twenty workgroups per compute unit.
template <auto Kernel>
inline uint32_t persistent_grid(int threads) {
  constexpr int kDevices = 64;
  static std::atomic<uint32_t> known[kDevices];
  int dev = 0, cus = 0, per = 0;
  const bool have_dev = hipGetDevice(&dev) == hipSuccess;
  const bool cached = have_dev && dev >= 0 && dev < kDevices;
  if (cached)
    if (const uint32_t g = known[dev].load(std::memory_order_relaxed)) return g;
  if (!have_dev || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, Kernel, threads, 0) != hipSuccess || per < 1) per = 1;
  const uint32_t g = std::max((uint32_t)(cus * per) / kQueueLanes * kQueueLanes, (uint32_t)kQueueLanes);
  if (cached) known[dev].store(g, std::memory_order_relaxed);
  return g;
}

// Grid schedule (P = false): a workgroup per work item, `items` of them at
// most.  Persistent: the device's resident workgroups.
template <bool P, auto Kernel, class... A>
inline void launch_items(uint32_t items, int threads, hipStream_t st, A... args) {
  Kernel<<<P ? persistent_grid<Kernel>(threads) : items, threads, 0, st>>>(args...);
}

}  // namespace gsr
