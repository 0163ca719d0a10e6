// Forward compositing: front-to-back alpha blending of each tile's sorted
// list, with per-pixel early termination once transmittance would fall
// below 1e-4.
//
// Every wave owns one 8 x 8 pixel block, one pixel per lane, and walks its
// tile's list by itself: no barrier, so a block stops as soon as its own 64
// pixels have.  Per 64 list entries each lane tests one record against the
// block (its falloff can reach alpha >= 1/255 there, tile_reaches), and the
// lanes whose record can put it behind those of the lanes below them in the
// wave's part of LDS; ids are loaded two, payloads one step ahead.  The wave
// then reads the kept records as broadcasts, four at a time: the four alphas
// are independent, and only T's multiply, compare and select chain from entry
// to entry.  VALU issue bounds it where the launch fills the chip (229M
// instructions on six 1600x900 views of 1M Gaussians: 347 us, 385 with the
// records staged by a tile's workgroup and one entry at a time), the chain of
// the longest list where it does not (64x48 with 2,000 Gaussians: 44 us, 234).
//
// Per pixel the kernel keeps T, the colour and the position one past the
// last composited entry, which the backward pass starts from.  With a
// target image the L1 loss is fused into the epilogue: dL/dimage per pixel
// and |image - target| summed per workgroup (a fixed butterfly per wave, then
// the waves in order), one partial per work item, added up in item order by
// k_l1_sum.
#include "kernels.hpp"
#include "raster.hpp"
#include "util.hpp"

namespace gsr {

// A wave's kept records of one step, in list order: (i0, j0, offx, offy),
// (qa, qb, qc, opacity), (r, g, b, list position + 1).  Room for the last
// group to be filled up with records of opacity zero.
constexpr int kFwdGroup = 4;
struct FwdStage {
  float4 rec[kWave + kFwdGroup - 1][3];
};

// A lane's pixel.  thr: the alpha from which it composites, 2 once it has
// stopped (or lies outside the image).
struct FwdPixel {
  float fx, fy, thr, T, C0, C1, C2;
  uint32_t last, cnt;
};

// G records from LDS.  Two ways to composite them, of the same results where
// the colours are finite (a weight of zero makes NaN of an infinite one, so
// steps that hold one take the second way): four at a time with selects only, so nothing stands between the alphas and
// T's chain (84 VGPRs, six waves per SIMD), for launches that cannot fill the
// chip with waves, whose time is the longest lists' latency; or two at a time
// with the lanes that do not composite switched off (five VALU instructions
// fewer per entry, 62 VGPRs, eight waves), for the others.
template <int G>
__device__ __forceinline__ void fwd_group(const float4 (*rec)[3], FwdPixel &s) {
  float4 a[G], b[G], c[G];
#pragma unroll
  for (int k = 0; k < G; ++k) {
    a[k] = rec[k][0];
    b[k] = rec[k][1];
    c[k] = rec[k][2];
  }
  float alpha[G];
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const float dx = (s.fx - a[k].x) - a[k].z;
    const float dy = (s.fy - a[k].y) - a[k].w;
    const float u = fmaf(b[k].y, dy, dx);
    const float q = fmaf(b[k].x, u * u, b[k].z * (dy * dy));
    alpha[k] = fminf(kAlphaMax, b[k].w * __builtin_amdgcn_exp2f(q));
  }
  if (G < kFwdGroup) {
#pragma unroll
    for (int k = 0; k < G; ++k) asm volatile("" : "+v"(alpha[k]));  // all alphas before the branches
#pragma unroll
    for (int k = 0; k < G; ++k) {
      if (alpha[k] >= s.thr) {
        asm volatile("");  // a branch, not selects
        const float tn = s.T * (1.0f - alpha[k]);
        if (tn < kTMin) {  // stop before the entry that would take T below 1e-4
          asm volatile("");
          s.thr = 2.0f;
        } else {
          const float w = alpha[k] * s.T;
          s.C0 = fmaf(w, c[k].x, s.C0);
          s.C1 = fmaf(w, c[k].y, s.C1);
          s.C2 = fmaf(w, c[k].z, s.C2);
          s.T = tn;
          s.last = __float_as_uint(c[k].w);
          s.cnt += 1u;
        }
      }
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const bool hit = alpha[k] >= s.thr;
    const float ah = hit ? alpha[k] : 0.0f;
    const float tn = s.T * (1.0f - ah);
    const bool stop = tn < kTMin;  // an entry that does not hit leaves tn = T
    const bool comp = hit & !stop;
    const float w = comp ? ah * s.T : 0.0f;
    s.C0 = fmaf(w, c[k].x, s.C0);
    s.C1 = fmaf(w, c[k].y, s.C1);
    s.C2 = fmaf(w, c[k].z, s.C2);
    s.T = stop ? s.T : tn;
    s.thr = stop ? 2.0f : s.thr;
    s.last = comp ? __float_as_uint(c[k].w) : s.last;
    s.cnt += comp ? 1u : 0u;
  }
}

// Walk of one wave's block at (bx, by) of a tile, G records at a time.
template <int TS, int G>
__device__ __forceinline__ void fwd_block(const ViewInfo *__restrict__ views, const Ws &ws, const Sizes &sz,
                                          uint32_t tile, int bx, int by, FwdStage &L, float *__restrict__ image,
                                          float *__restrict__ t_final, uint32_t *__restrict__ last_pos,
                                          uint32_t *__restrict__ n_contrib, const LossArgs &la, float &acc) {
  const ViewInfo vi = views[wave_view_of_tile(views, sz.n_views, tile)];
  const uint32_t lt = tile - vi.tile_base;
  const int ox = (int)(lt % (uint32_t)vi.tiles_x) * TS + bx, oy = (int)(lt / (uint32_t)vi.tiles_x) * TS + by;
  if (ox >= vi.w || oy >= vi.h) return;  // the block lies outside a ragged edge
  const uint32_t start = ws.tile_start[tile], n = ws.tile_count[tile];
  const uint32_t nrec = ws.scalars[kNumRecords];
  const int lane = lane_id();
  const int px = ox + (lane & 7), py = oy + (lane >> 3);
  const bool inside = px < vi.w && py < vi.h;
  FwdPixel s{(float)px, (float)py, inside ? kAlphaMin : 2.0f, 1.0f, 0.0f, 0.0f, 0.0f, 0u, 0u};

  const uint32_t *list = ws.tile_recs + start;
  auto ids = [&](uint32_t b) {
    const uint32_t i = b + (uint32_t)lane;
    uint32_t rec = i < n ? list[i] : 0u;
    if (rec >= nrec) {  // corrupt list (or no record at all): flag it, stay in bounds
      if (i < n) ws.scalars[kOverflow] = 4u;
      rec = 0;
    }
    return rec;
  };
  uint32_t rec = ids(0), rec_n = ids(kWave);
  float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0, p2 = p0;
  float p3 = 0.0f;
  auto payload = [&](uint32_t r) {
    const float4 *src = ws.rec_payload + (size_t)r * 4;
    p0 = src[0];
    p1 = src[1];
    p2 = src[2];
    p3 = src[3].x;
  };
  if (n > 0) payload(rec);
  for (uint32_t b0 = 0; b0 < n; b0 += kWave) {
    if (__ballot(s.thr < 1.0f) == 0) break;
    const bool keep = b0 + (uint32_t)lane < n && tile_reaches(p0, p1, p2, (float)ox, (float)oy, 8.0f);
    const uint64_t mask = __ballot(keep);
    const int kept = __popcll(mask);
    const bool odd = G > 2 && __ballot(keep && !(fabsf(p2.z) + fabsf(p2.w) + fabsf(p3) < INFINITY)) != 0;
    __builtin_amdgcn_wave_barrier();
    if (keep) {
      float4 *dst = L.rec[__popcll(mask & lanemask_lt())];
      dst[0] = make_float4(p0.x, p0.z, p1.x, p1.y);
      dst[1] = make_float4(p1.z, p1.w, p2.x, p2.y);
      dst[2] = make_float4(p2.z, p2.w, p3, __uint_as_float(b0 + (uint32_t)lane + 1u));
    }
    if (lane < G - 1) {
      float4 *dst = L.rec[kept + lane];
      dst[0] = dst[1] = dst[2] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __builtin_amdgcn_wave_barrier();
    rec = rec_n;
    if (b0 + kWave < n) {
      payload(rec);
      rec_n = ids(b0 + 2 * kWave);
    }
    if (G > 2 && odd) {
      for (int k = 0; k < kept; k += 2) fwd_group<2>(L.rec + k, s);
      continue;
    }
    for (int k = 0; k < kept; k += G) {
      fwd_group<G>(L.rec + k, s);
      if (__ballot(s.thr < 1.0f) == 0) break;
    }
  }

  if (inside) {
    const float T = s.T;
    const uint32_t hw = (uint32_t)vi.w * (uint32_t)vi.h;
    const uint32_t pixi = (uint32_t)py * (uint32_t)vi.w + (uint32_t)px;
    float *img = image + (size_t)3 * vi.pix_off;
    const float c0 = s.C0 + T * sz.bg[0], c1 = s.C1 + T * sz.bg[1], c2 = s.C2 + T * sz.bg[2];
    img[pixi] = c0;
    img[hw + pixi] = c1;
    img[2 * hw + pixi] = c2;
    if (la.target) {
      const float *tg = la.target + (size_t)3 * vi.pix_off;
      float *dl = la.dl + (size_t)3 * vi.pix_off;
      const float d0 = c0 - tg[pixi], d1 = c1 - tg[hw + pixi], d2 = c2 - tg[2 * hw + pixi];
      auto sgn = [&](float d) { return d > 0.0f ? la.inv_n : (d < 0.0f ? -la.inv_n : 0.0f); };
      dl[pixi] = sgn(d0);
      dl[hw + pixi] = sgn(d1);
      dl[2 * hw + pixi] = sgn(d2);
      acc += (fabsf(d0) + fabsf(d1)) + fabsf(d2);
    }
    t_final[vi.pix_off + pixi] = T;
    last_pos[vi.pix_off + pixi] = s.last;
    n_contrib[vi.pix_off + pixi] = s.cnt;
  }
}

// The fused loss keeps one partial per work item, so its fixed-order sum does
// not depend on which workgroup took which item: a butterfly per wave, then
// the wave that finishes last adds the waves' sums in order.  done: LDS, zero
// between items.
template <int NW>
__device__ __forceinline__ void item_loss(const LossArgs &la, float acc, float *red, uint32_t *done, uint32_t item) {
  if (!la.target) return;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, kWave);
  if (lane_id() == 0) {
    volatile float *r = red;
    r[wave_id()] = acc;
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the sum is in LDS before the count says so
    if (atomicAdd(done, 1u) == NW - 1u) {
      float s = r[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += r[w];
      la.part[item] = s;
      *done = 0u;
    }
  }
}

// A work item is a tile, walked by a workgroup with a wave per 8 x 8 block;
// at 8 px it is four tiles, a wave each.  Longest lists first.
template <int TS>
struct FwdItem {
  static constexpr int NW = TS == 32 ? 16 : 4;
};

template <int TS, bool P, int G>
__global__ __launch_bounds__(FwdItem<TS>::NW * 64) void k_raster_fwd(
    const ViewInfo *__restrict__ views, Ws ws, Sizes sz, float *__restrict__ image, float *__restrict__ t_final,
    uint32_t *__restrict__ last_pos, uint32_t *__restrict__ n_contrib, LossArgs la) {
  constexpr int NW = FwdItem<TS>::NW, TPI = TS == 8 ? 4 : 1;  // tiles per item
  __shared__ FwdStage S[NW];
  __shared__ float red[NW];
  __shared__ uint32_t take, done;
  if (ws.scalars[kOverflow]) return;
  if (threadIdx.x == 0) done = 0u;
  __syncthreads();
  const uint32_t n_items = (sz.t_tot + TPI - 1u) / TPI;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave_id());
  ItemQueue<P> q(ws.queues);
  for (uint32_t it = blockIdx.x; it < n_items; it = q.next(&take)) {
    float acc = 0.0f;
    const uint32_t i = TS == 8 ? it * 4u + w : it;
    if (i < sz.t_tot) {
      const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)ws.tile_order[i]);
      constexpr uint32_t NB = TS / 8;  // blocks per row of the tile
      const int bx = TS == 8 ? 0 : (int)(w % NB) * 8, by = TS == 8 ? 0 : (int)(w / NB) * 8;
      fwd_block<TS, G>(views, ws, sz, tile, bx, by, S[w], image, t_final, last_pos, n_contrib, la, acc);
    }
    item_loss<NW>(la, acc, red, &done, it);
  }
}

// Work items, and loss partials, of the forward.
uint32_t raster_fwd_grid(const Sizes &sz) { return sz.ts == 8 ? (sz.t_tot + 3u) / 4u : sz.t_tot; }

// Waves up to which a launch takes the group of four records: at 22,800 waves
// of long street lists four take 143 us and two 176, at 34,800 294 and 363,
// at 45,600 197 and 185 and at 136,800 400 and 347.
constexpr uint64_t kFwdFewWaves = 40960;

void launch_raster_fwd(const ViewInfo *views, const Ws &ws, const Sizes &sz, float *image, float *t_final,
                       uint32_t *last_pos, uint32_t *n_contrib, const LossArgs &la, hipStream_t st) {
  if (sz.t_tot == 0) return;
  const bool few = (uint64_t)sz.t_tot * (uint64_t)(sz.ts * sz.ts / 64) <= kFwdFewWaves;
#define FWD(TS, P, G)                                                                                             \
  launch_items<P, k_raster_fwd<TS, P, G>>(raster_fwd_grid(sz), FwdItem<TS>::NW * 64, st, views, ws, sz, image,    \
                                          t_final, last_pos, n_contrib, la)
#define FWD_TS(TS)                                    \
  if (sz.persistent) {                                \
    if (few) FWD(TS, true, 4); else FWD(TS, true, 2); \
  } else {                                            \
    if (few) FWD(TS, false, 4); else FWD(TS, false, 2); \
  }
  switch (sz.ts) {
    case 8: FWD_TS(8) break;
    case 32: FWD_TS(32) break;
    default: FWD_TS(16) break;
  }
#undef FWD_TS
#undef FWD
}

}  // namespace gsr
