// Runs the binning on records of the caller's, past the preprocessing that
// writes them, in a plan of t_tot tiles and the given capacities.  A record is
// its tile rectangle (tx0 | tx1 << 16, ty0 | ty1 << 16, first tile, row pitch).
// out: the overflow code, then the list lengths.  Returns a HIP status.
#include <hip/hip_runtime.h>

#include <vector>

#include "kernels.hpp"

using namespace gsr;

namespace {
struct Buffers {
  std::vector<void *> all;
  ~Buffers() {
    for (void *p : all) (void)hipFree(p);
  }
  template <class T>
  T *take(size_t n) {
    void *p = nullptr;
    if (hipMalloc(&p, n * sizeof(T) + 256) != hipSuccess) return nullptr;
    all.push_back(p);
    return static_cast<T *>(p);
  }
};
}  // namespace

extern "C" int run_binning(uint32_t t_tot, uint32_t cap_rec, uint32_t cap_pairs, uint32_t n_rec, const uint4 *rects,
                           uint32_t *out) {
  if (n_rec > cap_rec) return -1;
  Sizes sz{};
  sz.n = cap_rec;
  sz.n_views = 1;
  sz.ts = 16;
  sz.t_tot = t_tot;
  sz.cap_rec = cap_rec;
  sz.cap_pairs = cap_pairs;
  sz.long_list = kLongAuto;
  const BinningScratch bs = binning_scratch(sz);
  Buffers b;
  Ws ws{};
  ws.scalars = b.take<uint32_t>(kNumScalars);
  ws.tile_count = b.take<uint32_t>(t_tot);
  ws.tile_start = b.take<uint32_t>(t_tot);
  ws.tile_order = b.take<uint32_t>(t_tot);
  ws.tile_tmp = b.take<uint32_t>(2 * (size_t)t_tot);
  ws.rec_rect = b.take<uint4>(cap_rec);
  ws.rec_tmp = b.take<uint32_t>(5 * (size_t)cap_rec);
  ws.radix_hist = b.take<uint32_t>(bs.radix_hist);
  ws.scan_part = b.take<uint32_t>(bs.scan_part);
  ws.pairs_tmp = b.take<uint32_t>(2 * (size_t)cap_pairs);
  ws.tile_recs = b.take<uint32_t>(cap_pairs);
  ws.partials = b.take<float>(9 * (size_t)cap_pairs + 12 * (size_t)cap_rec);
  if (b.all.size() != 12) return -2;
  std::vector<uint32_t> scalars(kNumScalars), perm(n_rec), area(n_rec), zero(t_tot);
  for (uint32_t i = 0; i < n_rec; ++i) {
    perm[i] = i;
    area[i] = ((rects[i].x >> 16) - (rects[i].x & 0xFFFFu) + 1) * ((rects[i].y >> 16) - (rects[i].y & 0xFFFFu) + 1);
    scalars[kNumPairs] += area[i];
  }
  if (scalars[kNumPairs] > cap_pairs) return -3;
  scalars[kNumRecords] = n_rec;
  hipError_t e = hipSuccess;
  auto up = [&](void *d, const void *s, size_t n) {
    if (e == hipSuccess) e = hipMemcpy(d, s, n, hipMemcpyHostToDevice);
  };
  up(ws.scalars, scalars.data(), kNumScalars * 4);
  up(ws.tile_count, zero.data(), t_tot * 4);
  up(ws.tile_start, zero.data(), t_tot * 4);
  up(ws.rec_tmp + cap_rec, perm.data(), n_rec * 4);
  up(ws.rec_tmp + 4 * (size_t)cap_rec, area.data(), n_rec * 4);
  up(ws.rec_rect, rects, n_rec * 16);
  up(ws.partials, rects, n_rec * 16);  // in depth order
  if (e != hipSuccess) return e;
  launch_binning(nullptr, ws, sz, nullptr);
  e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(scalars.data(), ws.scalars, kNumScalars * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(out + 1, ws.tile_count, t_tot * 4, hipMemcpyDeviceToHost);
  out[0] = scalars[kOverflow];
  return e;
}
