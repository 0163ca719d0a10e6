// Backward compositing: the adjoint of the forward blend, walking each
// tile's list back to front.
//
// Per pixel the walk starts at the stored end position with T = T_final and
// S = sum_ch g_ch bg_ch, the suffix colour's product with the pixel's
// gradient g (one value per pixel where the suffix colour took three).  For
// every entry it recomputes alpha exactly as the forward did, recovers the
// transmittance in front of it by division, T_i = T_{i+1} / (1 - alpha_i), and
// accumulates
//   dL/drgb   += g alpha T_i
//   dL/dalpha  = T_i (sum_ch g_ch rgb_ch - S),  S <- S + alpha (sum_ch g_ch rgb_ch - S)
// and, unless alpha hit the 0.99 cap, dL/dopacity and dL/dq through
// alpha = opacity 2^q, then dL/d(qa, qb, qc, offx, offy) through q.
//
// Records whose alpha >= 1/255 ellipse misses the tile (or, with a wave per
// block, the block) are not visited.  The 9 per-entry sums are reduced over
// each wave (skipped when no lane of the wave composited the entry), combined
// over the waves in LDS, and written once per (record, tile) into that pair's
// slot -- no floating-point atomics, so the result is deterministic.  The
// transmittance is recovered with the hardware reciprocal (1 ulp), which
// keeps the accumulated relative error of T near 1e-6 over a few hundred
// entries.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "raster.hpp"
#include "util.hpp"

namespace gsr {

constexpr float kLn2 = 0x1.62e43p-1f;

// A pair's nine partial gradients, packed at slot * 9 (36 bytes, so only
// 4-byte aligned).
__device__ __forceinline__ void store_partial(const Ws &ws, uint32_t slot, const float (&v)[9]) {
  float *dst = ws.partials + (size_t)slot * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) dst[k] = v[k];
}

__device__ __forceinline__ void store_zero_partial(const Ws &ws, uint32_t slot) {
  const float z[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  store_partial(ws, slot, z);
}

// Barrier over the threads that share one tile's LDS: the workgroup, or a
// single wave (whose LDS accesses are performed in order).
template <bool WG>
__device__ __forceinline__ void group_sync() {
  if (WG) {
    __syncthreads();
  } else {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
  }
}

// A pair's payload gradients from its nine pixel sums (dq u, dq dy, dq u^2,
// dq u dy, dq dy^2, dq, and w g of the three channels):
//   q = qa u^2 + qc dy^2, u = dx + qb dy, dx = ... - offx, dy = ... - offy:
//   dL/dqb = 2 qa sum(dq u dy),  dL/doffx = -2 qa sum(dq u),
//   dL/doffy = -(2 qa qb sum(dq u) + 2 qc sum(dq dy))   (times ln 2)
//   dL/dopacity = sum(dq) / opacity, as alpha = opacity 2^q
// conic: (qa, qb, qc, opacity).
__device__ __forceinline__ void store_gradients(const Ws &ws, uint32_t slot, const float (&s9)[9], const float4 conic) {
  const float qa2 = 2.0f * conic.x, qc2 = 2.0f * conic.z;
  const float d_offx = -qa2 * s9[0], d_offy = -fmaf(qa2 * conic.y, s9[0], qc2 * s9[1]);
  const float v[9] = {d_offx * kLn2,   d_offy * kLn2, s9[2] * kLn2, qa2 * s9[3] * kLn2, s9[4] * kLn2,
                      s9[5] / conic.w, s9[6],         s9[7],        s9[8]};
  store_partial(ws, slot, v);
}

// What a walk needs of its tile: the view, the list and its place.
struct BwdTile {
  uint32_t tx, ty, start, n, nrec;
  float k0, k1, k2;  // the colours' origin
  ViewInfo vi;
};

__device__ __forceinline__ float wave_first(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

template <int TS>
__device__ __forceinline__ BwdTile bwd_tile(const ViewInfo *__restrict__ views, const Ws &ws, const Sizes &sz, uint32_t tile) {
  BwdTile b;
  b.vi = views[wave_view_of_tile(views, sz.n_views, tile)];
  const uint32_t lt = tile - b.vi.tile_base;
  b.tx = lt % (uint32_t)b.vi.tiles_x;
  b.ty = lt / (uint32_t)b.vi.tiles_x;
  b.start = ws.tile_start[tile];
  b.n = ws.tile_count[tile];
  b.nrec = ws.scalars[kNumRecords];
  // Colours are counted from that of the list's first entry (in [0, 1]): the
  // differences that the walk forms do not depend on the origin, but their
  // rounding does (opacity gradients of three street scenes are off their 64
  // bit values by 2.70e-7 from black, 2.44e-7 from here, 2.54e-7 with three
  // suffix colours).
  b.k0 = b.k1 = b.k2 = 0.0f;
  if (b.n) {
    const uint32_t rec = (uint32_t)__builtin_amdgcn_readfirstlane((int)ws.tile_recs[b.start]);
    const float *f = reinterpret_cast<const float *>(ws.rec_payload + (size_t)(rec < b.nrec ? rec : 0u) * 4);
    b.k0 = wave_first(fminf(fmaxf(f[10], 0.0f), 1.0f));
    b.k1 = wave_first(fminf(fmaxf(f[11], 0.0f), 1.0f));
    b.k2 = wave_first(fminf(fmaxf(f[12], 0.0f), 1.0f));
  }
  return b;
}

// Slot of the tile's pair of record rec in the record-major partials array; a
// record out of range is flagged and replaced by record 0.
__device__ __forceinline__ uint32_t pair_slot(const Ws &ws, const BwdTile &b, uint32_t &rec) {
  if (rec >= b.nrec) {  // corrupt list: flag it, stay in bounds
    ws.scalars[kOverflow] = 4u;
    rec = 0;
  }
  const uint4 rc = ws.rec_rect[rec];
  const uint32_t tx0 = rc.x & 0xFFFFu, tx1 = rc.x >> 16, ty0 = rc.y & 0xFFFFu, ty1 = rc.y >> 16;
  if (b.tx < tx0 || b.tx > tx1 || b.ty < ty0 || b.ty > ty1) {  // not this record's tile: corrupt list
    ws.scalars[kOverflow] = 4u;
    return ws.rec_pairoff[rec];
  }
  return ws.rec_pairoff[rec] + (b.ty - ty0) * (tx1 - tx0 + 1) + (b.tx - tx0);
}

// One pixel's state: T behind the walk, its image gradient, S, and the end of
// its list.
struct BwdPixel {
  float fx, fy, T, g0, g1, g2, S;
  uint32_t last;
};

__device__ __forceinline__ BwdPixel bwd_pixel(const BwdTile &b, const Sizes &sz, int px, int py,
                                              const float *__restrict__ t_final, const uint32_t *__restrict__ last_pos,
                                              const float *__restrict__ dL_dimage) {
  BwdPixel p{(float)px, (float)py, 1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0u};
  if (px < b.vi.w && py < b.vi.h) {
    const uint32_t hw = (uint32_t)b.vi.w * (uint32_t)b.vi.h;
    const uint32_t pixi = (uint32_t)py * (uint32_t)b.vi.w + (uint32_t)px;
    p.T = t_final[b.vi.pix_off + pixi];
    p.last = last_pos[b.vi.pix_off + pixi];
    const float *gi = dL_dimage + (size_t)3 * b.vi.pix_off;
    p.g0 = gi[pixi];
    p.g1 = gi[hw + pixi];
    p.g2 = gi[2 * hw + pixi];
  }
  p.S = fmaf(p.g0, sz.bg[0] - b.k0, fmaf(p.g1, sz.bg[1] - b.k1, p.g2 * (sz.bg[2] - b.k2)));
  return p;
}

// ---- a 16 x 16 tile by one wave -------------------------------------------
// Four 8 x 8 blocks, one pixel of each per lane, so a record's wave reduction
// is paid once for all four.  Lane j holds record j of a 64-record batch: it
// tests the record against the tile (tile_reaches) and the blocks' boxes, the
// ballots of which are the records to visit per block, and writes its
// gradients at the end.
struct BwdWaveLds {
  float4 rec[kWave][3];  // (i0, j0, offx, offy), (qa, qb, qc, opacity), (r, g, b, -)
  float g[kWave * 9];
};

__device__ __forceinline__ void bwd_wave(const ViewInfo *__restrict__ views, const Ws &ws, const Sizes &sz, uint32_t tile,
                                         BwdWaveLds &L, const float *__restrict__ t_final,
                                         const uint32_t *__restrict__ last_pos, const float *__restrict__ dL_dimage) {
  const BwdTile b = bwd_tile<16>(views, ws, sz, tile);
  if (b.n == 0) return;
  const int lane = lane_id(), mine = sum9_value(lane);
  const int ox = (int)b.tx * 16, oy = (int)b.ty * 16;
  BwdPixel px[4];
  uint32_t end[4], max_last = 0;  // per block, the end of its longest pixel's walk
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    px[p] = bwd_pixel(b, sz, ox + (lane & 7) + (p & 1) * 8, oy + (lane >> 3) + (p >> 1) * 8, t_final, last_pos, dL_dimage);
    end[p] = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_reduce_max(px[p].last));
    max_last = max(max_last, end[p]);
  }
  // entries no pixel reaches get zero gradients
  for (uint32_t i = max_last + (uint32_t)lane; i < b.n; i += kWave) {
    uint32_t rec = ws.tile_recs[b.start + i];
    store_zero_partial(ws, pair_slot(ws, b, rec));
  }
  // batches walk the list backwards; the next (earlier) batch is fetched into
  // registers while the current one is processed
  float4 f0, f1, f2;
  float f3 = 0.0f;
  uint32_t fslot = 0;
  f0 = f1 = f2 = make_float4(0.f, 0.f, 0.f, 0.f);
  auto fetch = [&](uint32_t lo, uint32_t hi) {
    if (lo + (uint32_t)lane < hi) {
      uint32_t rec = ws.tile_recs[b.start + lo + (uint32_t)lane];
      fslot = pair_slot(ws, b, rec);
      const float4 *src = ws.rec_payload + (size_t)rec * 4;
      f0 = src[0];
      f1 = src[1];
      f2 = src[2];
      f3 = src[3].x;
    }
  };
  auto batch_lo = [](uint32_t hi) { return hi > (uint32_t)kWave ? hi - kWave : 0u; };
  fetch(batch_lo(max_last), max_last);
  for (uint32_t hi = max_last; hi > 0;) {
    const uint32_t lo = batch_lo(hi), m = hi - lo;
    group_sync<false>();
    const bool live = (uint32_t)lane < m;
    const uint32_t slot = fslot;
    uint64_t mk[4];
    {
      const bool keep = live && tile_reaches(f0, f1, f2, (float)ox, (float)oy, 16.0f);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float bx = (float)(ox + (p & 1) * 8), by = (float)(oy + (p >> 1) * 8);
        mk[p] = __ballot(keep & (lo + (uint32_t)lane < end[p]) & (f0.x <= bx + 7.0f) & (f0.y >= bx) &
                         (f0.z <= by + 7.0f) & (f0.w >= by));
      }
    }
    L.rec[lane][0] = make_float4(f0.x, f0.z, f1.x, f1.y);
    L.rec[lane][1] = make_float4(f1.z, f1.w, f2.x, f2.y);
    L.rec[lane][2] = make_float4(f2.z - b.k0, f2.w - b.k1, f3 - b.k2, 0.0f);
    fetch(batch_lo(lo), lo);
    group_sync<false>();
    uint64_t hit = 0;  // records some pixel composited
    for (uint64_t rem = (mk[0] | mk[1]) | (mk[2] | mk[3]); rem;) {
      const int j = 63 - __builtin_clzll(rem);
      const uint64_t bit = uint64_t(1) << j;
      rem &= ~bit;
      const uint32_t pos = lo + (uint32_t)j;
      const float4 q0 = L.rec[j][0], q1 = L.rec[j][1], q2 = L.rec[j][2];
      // Per 8 x 8 block, the lanes that composite.  With dq = dL/dalpha alpha
      // (dL/dq without the ln 2 of d alpha / dq) each adds dq u, dq dy,
      // dq u^2, dq u dy, dq dy^2, dq and w g.  The empty asm keeps the zeros
      // opaque, so the compiler does not re-materialise them on every path.
      float a_u = 0.f, a_dy = 0.f, a_qa = 0.f, a_udy = 0.f, a_qc = 0.f, a_q = 0.f, a_r = 0.f, a_g = 0.f, a_b = 0.f;
      asm volatile("" : "+v"(a_u), "+v"(a_dy), "+v"(a_qa), "+v"(a_udy), "+v"(a_qc), "+v"(a_q), "+v"(a_r), "+v"(a_g),
                   "+v"(a_b));
      bool any = false;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        if (!(mk[p] & bit)) continue;  // uniform
        BwdPixel &s = px[p];
        const float dx = (s.fx - q0.x) - q0.z;
        const float dy = (s.fy - q0.y) - q0.w;
        const float u = fmaf(q1.y, dy, dx);
        const float u2 = u * u, dy2 = dy * dy;
        const float q = fmaf(q1.x, u2, q1.z * dy2);
        const float oe = q1.w * __builtin_amdgcn_exp2f(q);
        const float alpha = fminf(kAlphaMax, oe);
        const bool comp = (pos < s.last) & (alpha >= kAlphaMin);
        if (__ballot(comp) == 0) continue;  // uniform
        any = true;
        if (comp) {
          asm volatile("");  // lanes off, not selects
          const float ti = s.T * __builtin_amdgcn_rcpf(1.0f - alpha);
          const float w = alpha * ti;
          a_r = fmaf(s.g0, w, a_r);
          a_g = fmaf(s.g1, w, a_g);
          a_b = fmaf(s.g2, w, a_b);
          const float d = fmaf(s.g0, q2.x, fmaf(s.g1, q2.y, s.g2 * q2.z)) - s.S;
          s.S = fmaf(alpha, d, s.S);
          s.T = ti;
          if (oe <= kAlphaMax) {  // at the 0.99 cap alpha's derivative is zero
            const float dq = ti * d * alpha;
            a_q += dq;
            const float du = dq * u;
            a_u += du;
            a_dy = fmaf(dq, dy, a_dy);
            a_qa = fmaf(dq, u2, a_qa);
            a_udy = fmaf(du, dy, a_udy);
            a_qc = fmaf(dq, dy2, a_qc);
          }
        }
      }
      if (any) {
        hit |= bit;
        const float v9[9] = {a_u, a_dy, a_qa, a_udy, a_qc, a_q, a_r, a_g, a_b};
        const float sum = wave_sum9_packed(v9);
        if (mine >= 0) L.g[j * 9 + mine] = sum;
      }
    }
    group_sync<false>();
    if (live) {
      if ((hit >> lane) & 1u) {
        float s9[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) s9[c] = L.g[lane * 9 + c];
        store_gradients(ws, slot, s9, L.rec[lane][1]);
      } else {
        store_zero_partial(ws, slot);
      }
    }
    hi = lo;
  }
}

// w g, and 0 for w = 0 also where g is not finite (v_mul_legacy_f32).
__device__ __forceinline__ float zero_mul(float w, float g) {
  float r;
  asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(w), "v"(g));
  return r;
}

// ---- a tile by a wave per 8 x 8 block -------------------------------------
// For long lists, whose time is the chain of their records: NW waves share
// B-record batches, a wave visits only the records whose falloff reaches its
// own block (tile_reaches, a ballot per 64 records) and that lie before the
// end of its own pixels' walks, G at a time: alphas and reductions of the G
// records overlap, only T and S chain from record to record.  One view of the
// rig, whose backward is its longest list: 640 us with one record at a time
// under two branches, 440 now; 64x48 with 2,000 Gaussians 411 and 112.
// Lanes that do not composite take alpha = 0, which leaves T (rcp(1) = 1), S
// and every sum as they are, also where the pixel's gradient is not finite (S
// is not then either).  A colour that is not finite would reach S by 0 times
// infinity: in batches that hold one, or one of 2^40 and more, such lanes take
// 0 for the colour product (six 800x450 views of 300k Gaussians 312 us without
// this, 316 with it, 321 with the select in every batch).
template <int B, int NW>
struct BwdBlockLds {
  float4 box[B];
  float4 rec[B + 1][3];   // as above; rec[B] has opacity zero, for a group's missing records
  float g[NW][B][9];      // the waves' sums of the records they visited
  uint64_t seen[NW][B / kWave];
  uint32_t huge[B / kWave];  // of 64 records each: a colour whose product with a gradient may be infinite
  uint32_t red[NW];
};

template <int TS, int NW, int B, int G>
__device__ __forceinline__ void bwd_block(const ViewInfo *__restrict__ views, const Ws &ws, const Sizes &sz, uint32_t tile,
                                          int t, BwdBlockLds<B, NW> &L, const float *__restrict__ t_final,
                                          const uint32_t *__restrict__ last_pos, const float *__restrict__ dL_dimage) {
  constexpr bool WG = NW > 1;
  constexpr uint32_t NT = NW * kWave;
  constexpr int NC = B / kWave, NB = TS / 8;
  const BwdTile b = bwd_tile<TS>(views, ws, sz, tile);
  if (b.n == 0) return;
  const int lane = lane_id(), wv = WG ? (int)__builtin_amdgcn_readfirstlane(t / kWave) : 0, mine = sum9_value(lane);
  const int ox = (int)b.tx * TS + (wv % NB) * 8, oy = (int)b.ty * TS + (wv / NB) * 8;
  BwdPixel s = bwd_pixel(b, sz, ox + (lane & 7), oy + (lane >> 3), t_final, last_pos, dL_dimage);
  const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_reduce_max(s.last));
  uint32_t max_last = end;
  if (WG) {
    if (lane == 0) L.red[wv] = end;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) max_last = max(max_last, L.red[w]);
    max_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)max_last);
  }
  if (t < 3) L.rec[B][t] = make_float4(0.f, 0.f, 0.f, 0.f);
  // entries no pixel reaches get zero gradients
  for (uint32_t i = max_last + (uint32_t)t; i < b.n; i += NT) {
    uint32_t rec = ws.tile_recs[b.start + i];
    store_zero_partial(ws, pair_slot(ws, b, rec));
  }
  float4 f0, f1, f2;
  float f3 = 0.0f;
  uint32_t fslot = 0;
  f0 = f1 = f2 = make_float4(0.f, 0.f, 0.f, 0.f);
  auto fetch = [&](uint32_t lo, uint32_t hi) {
    if ((uint32_t)t < B && lo + (uint32_t)t < hi) {
      uint32_t rec = ws.tile_recs[b.start + lo + (uint32_t)t];
      fslot = pair_slot(ws, b, rec);
      const float4 *src = ws.rec_payload + (size_t)rec * 4;
      f0 = src[0];
      f1 = src[1];
      f2 = src[2];
      f3 = src[3].x;
    }
  };
  auto batch_lo = [](uint32_t hi) { return hi > (uint32_t)B ? hi - B : 0u; };
  fetch(batch_lo(max_last), max_last);
  for (uint32_t hi = max_last; hi > 0;) {
    const uint32_t lo = batch_lo(hi), m = hi - lo;
    group_sync<WG>();
    const uint32_t slot = fslot;
    if ((uint32_t)t < m) {
      L.box[t] = f0;
      L.rec[t][0] = make_float4(f0.x, f0.z, f1.x, f1.y);
      L.rec[t][1] = make_float4(f1.z, f1.w, f2.x, f2.y);
      L.rec[t][2] = make_float4(f2.z - b.k0, f2.w - b.k1, f3 - b.k2, 0.0f);
    }
    if (wv < NC) {  // the waves that stage
      const uint64_t big = __ballot((uint32_t)t < m && !(fabsf(f2.z) + fabsf(f2.w) + fabsf(f3) < 0x1p40f));
      if (lane == 0) L.huge[wv] = big != 0;
    }
    fetch(batch_lo(lo), lo);
    group_sync<WG>();
    uint64_t mk[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const uint32_t j = (uint32_t)(c * kWave + lane);
      bool keep = j < m && lo + j < end;
      if (keep) {
        const float4 q0 = L.rec[j][0], q1 = L.rec[j][1];
        keep = tile_reaches(L.box[j], make_float4(q0.z, q0.w, q1.x, q1.y), make_float4(q1.z, q1.w, 0.f, 0.f), (float)ox,
                            (float)oy, 8.0f);
      }
      mk[c] = __ballot(keep);
      if (lane == 0) L.seen[wv][c] = mk[c];
    }
    auto visit = [&](int c, uint64_t rem, auto group, auto any_colour) {
      constexpr int N = decltype(group)::value;
      while (rem) {
        int j[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const int jb = 63 - __builtin_clzll(rem | 1u);
          j[k] = rem ? c * kWave + jb : B;  // (uniform) none left: the record of opacity zero
          rem &= ~(uint64_t(1) << jb);
        }
        float4 q0[N], q1[N], q2[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          q0[k] = L.rec[j[k]][0];
          q1[k] = L.rec[j[k]][1];
          q2[k] = L.rec[j[k]][2];
        }
        float u[N], dy[N], al[N], gc[N];
        bool free[N];  // composited below the 0.99 cap, where alpha's derivative is zero
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const float dx = (s.fx - q0[k].x) - q0[k].z;
          dy[k] = (s.fy - q0[k].y) - q0[k].w;
          u[k] = fmaf(q1[k].y, dy[k], dx);
          const float q = fmaf(q1[k].x, u[k] * u[k], q1[k].z * (dy[k] * dy[k]));
          const float oe = q1[k].w * __builtin_amdgcn_exp2f(q);
          const float alpha = fminf(kAlphaMax, oe);
          const bool comp = (lo + (uint32_t)j[k] < s.last) & (alpha >= kAlphaMin);
          al[k] = comp ? alpha : 0.0f;
          free[k] = comp & (oe <= kAlphaMax);
          gc[k] = fmaf(s.g0, q2[k].x, fmaf(s.g1, q2[k].y, s.g2 * q2[k].z));
          if (decltype(any_colour)::value) gc[k] = comp ? gc[k] : 0.0f;
        }
        float w[N], dq[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const float ti = s.T * __builtin_amdgcn_rcpf(1.0f - al[k]);
          w[k] = al[k] * ti;
          const float d = gc[k] - s.S;
          s.S = fmaf(al[k], d, s.S);
          s.T = ti;
          dq[k] = free[k] ? ti * d * al[k] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
          const float du = dq[k] * u[k], dd = dq[k] * dy[k];
          const float v9[9] = {du, dd, du * u[k], du * dy[k], dd * dy[k], dq[k],
                               zero_mul(w[k], s.g0), zero_mul(w[k], s.g1), zero_mul(w[k], s.g2)};
          const float sum = wave_sum9_packed(v9);
          if (mine >= 0 && j[k] < B) L.g[wv][j[k]][mine] = sum;
        }
      }
    };
    uint32_t huge = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) huge |= L.huge[c];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(huge) != 0, 0)) {
#pragma unroll
      for (int c = NC - 1; c >= 0; --c) visit(c, mk[c], std::integral_constant<int, G>(), std::true_type());
    } else {
#pragma unroll
      for (int c = NC - 1; c >= 0; --c) visit(c, mk[c], std::integral_constant<int, G>(), std::false_type());
    }
    group_sync<WG>();
    if ((uint32_t)t < m) {
      float s9[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) s9[c] = 0.0f;
      bool any = false;
#pragma unroll
      for (int w = 0; w < NW; ++w)
        if ((L.seen[w][t / kWave] >> lane) & 1u) {
          any = true;
#pragma unroll
          for (int c = 0; c < 9; ++c) s9[c] += L.g[w][t][c];
        }
      if (any)
        store_gradients(ws, slot, s9, L.rec[t][1]);
      else
        store_zero_partial(ws, slot);
    }
    hi = lo;
  }
}

// 16 px tiles.  The long lists (kNumLong of them, a prefix of the
// longest-first order; see k_tile_ranges) are one work item each, for the
// whole workgroup, a wave per block; the remaining tiles are items of four,
// one wave each, neighbours in the longest-first order having similar
// lengths.
union BwdLds16 {
  BwdBlockLds<128, 4> block;
  BwdWaveLds wave[4];
};

// VALU issue bounds it (416M instructions a launch on the rig, 529M when every
// lane kept three suffix colours, composited under selects and the wave sums
// took 33 instructions): six 1600x900 views of 1M Gaussians 643 us (785).  Five
// waves per SIMD and the blocks' masks from the boxes, from one build (rig; 40
// mixed views of 2M, two scenes; six 800x450 views of 300k, one long list):
//   as it is                            643 us  7.71 ms  6.43 ms  318 us
//   four waves                          642     7.67     6.57     318
//   six waves, 64-record batches        636     7.56     6.47     353
//   masks by tile_reaches per block     648     7.54     6.63     316
//   the same behind the tile's test     653     7.75     6.69     322
template <bool P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_raster_bwd16(
    const ViewInfo *__restrict__ views, Ws ws, Sizes sz, const float *__restrict__ t_final,
    const uint32_t *__restrict__ last_pos, const float *__restrict__ dL_dimage) {
  __shared__ BwdLds16 S;
  __shared__ uint32_t take;
  if (ws.scalars[kOverflow]) return;
  uint32_t *queue = ws.queues + kQueueLanes * kQueueStride;
  const uint32_t n_long = ws.scalars[kNumLong];
  const uint32_t n_items = n_long + (sz.t_tot - n_long + 3u) / 4u;
  const int t = threadIdx.x;
  ItemQueue<P> q(queue);
  for (uint32_t it = blockIdx.x; it < n_items; it = q.next(&take)) {
    if (it < n_long) {
      bwd_block<16, 4, 128, 2>(views, ws, sz, ws.tile_order[it], t, S.block, t_final, last_pos, dL_dimage);
    } else {
      const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave_id()), i = n_long + (it - n_long) * 4u + w;
      if (i < sz.t_tot) {
        const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)ws.tile_order[i]);
        bwd_wave(views, ws, sz, tile, S.wave[w], t_final, last_pos, dL_dimage);
      }
    }
  }
}

// A wave per 8 x 8 block for every tile, a tile per work item: 8 and 32 px,
// and 16 px launches of at most kFewTiles tiles whose lists are all long (by
// the library's choice, or long_list 0), which leave the chip room for batches
// of 256 records (54 KB of LDS; all four waves stage, half the barriers).  At
// 8 px four records at a time (921 us on the rig, two take 934; one under
// branches took 1016); at 32 px, where 16 waves share a tile, two and eight
// waves per SIMD (1331 us; four records and half the waves 1901; four waves of
// four blocks each 1667).  At 16 px this walk and the mixed one above: 64x48
// with 2,000 Gaussians (12 tiles) 103 and 110 us, 1280x720 with 300k (3,600)
// 178 and 191, 1600x900 with 300k (5,700) 147 and 158, 1920x1080 with 500k
// (8,160) 228 and 200; 128- and 192-record batches take 108 and 107 us on the
// first, eight records at a time 114.

template <int TS>
struct BwdItem {
  static constexpr int NW = (TS / 8) * (TS / 8), NT = NW * 64;
  static constexpr int G = TS == 32 ? 2 : 4, B = TS == 16 ? 256 : 64;
  static constexpr int kWaves = TS == 8 ? 5 : TS == 16 ? 3 : 8;
};

template <int TS, bool P>
__global__ __launch_bounds__(BwdItem<TS>::NT) __attribute__((amdgpu_waves_per_eu(BwdItem<TS>::kWaves))) void k_raster_bwd(
    const ViewInfo *__restrict__ views, Ws ws, Sizes sz, const float *__restrict__ t_final,
    const uint32_t *__restrict__ last_pos, const float *__restrict__ dL_dimage) {
  constexpr int NW = BwdItem<TS>::NW, B = BwdItem<TS>::B;
  __shared__ BwdBlockLds<B, NW> S;
  __shared__ uint32_t take;
  if (ws.scalars[kOverflow]) return;
  ItemQueue<P> q(ws.queues + kQueueLanes * kQueueStride);
  for (uint32_t i = blockIdx.x; i < sz.t_tot; i = q.next(&take))
    bwd_block<TS, NW, B, BwdItem<TS>::G>(views, ws, sz, ws.tile_order[i], threadIdx.x, S, t_final, last_pos, dL_dimage);
}

// Sum each record's per-tile partials (contiguous, record-major) into its
// reduced gradient.  Each wave takes 64 consecutive records: a lane sums a
// record of at most kBig pairs alone, two pairs per step so their loads
// overlap; larger footprints are summed by the whole wave (lane l takes
// pairs l, l + 64, ...) and reduced across lanes, so one big record does not
// hold its wave for hundreds of dependent loads.
constexpr uint32_t kBig = 16;

__device__ __forceinline__ void add_partial(const float *__restrict__ src, float (&v)[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) v[k] += src[k];
}

// step (optional): the Adam step counter, incremented here (before the
// per-Gaussian kernel that reads it) rather than by a launch of its own.  On
// a capacity overflow nothing is updated (the per-Gaussian kernel skips its
// Adam step too), so the counter stays with the moments.
__global__ __launch_bounds__(256) void k_reduce_pairs(Ws ws, int32_t *step) {
  // the next backward's work queue starts from zero
  if (blockIdx.x == 0 && threadIdx.x < kQueueLanes)
    ws.queues[(kQueueLanes + threadIdx.x) * kQueueStride] = 0u;
  if (ws.scalars[kOverflow]) return;
  if (step && blockIdx.x == 0 && threadIdx.x == 0) *step += 1;
  const uint32_t nrec = ws.scalars[kNumRecords];
  const int lane = lane_id(), mine = sum9_value(lane);
  const uint32_t wave_stride = gridDim.x * (blockDim.x / kWave) * kWave;
  for (uint32_t wbase = (blockIdx.x * (blockDim.x / kWave) + wave_id()) * kWave; wbase < nrec;
       wbase += wave_stride) {
    const uint32_t r = wbase + lane;
    uint32_t cnt = 0, p0 = 0;
    if (r < nrec) {
      const uint4 rc = ws.rec_rect[r];
      cnt = ((rc.x >> 16) - (rc.x & 0xFFFFu) + 1) * ((rc.y >> 16) - (rc.y & 0xFFFFu) + 1);
      p0 = ws.rec_pairoff[r];
    }
    if (r < nrec && cnt <= kBig) {
      float a[9], b[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) a[k] = b[k] = 0.0f;
      // even pairs into a, odd ones into b, in order; four pairs' loads are
      // issued before their sums
      uint32_t k = 0;
      for (; k + 3 < cnt; k += 4) {
        const float *src = ws.partials + (size_t)(p0 + k) * 9;
        float x[36];
#pragma unroll
        for (int c = 0; c < 36; ++c) x[c] = src[c];
#pragma unroll
        for (int c = 0; c < 9; ++c) {
          a[c] += x[c];
          b[c] += x[9 + c];
          a[c] += x[18 + c];
          b[c] += x[27 + c];
        }
      }
      for (; k + 1 < cnt; k += 2) {
        add_partial(ws.partials + (size_t)(p0 + k) * 9, a);
        add_partial(ws.partials + (size_t)(p0 + k + 1) * 9, b);
      }
      if (k < cnt) add_partial(ws.partials + (size_t)(p0 + k) * 9, a);
#pragma unroll
      for (int c = 0; c < 9; ++c) a[c] += b[c];
      ws.g2d[(size_t)r * 3 + 0] = make_float4(a[0], a[1], a[2], a[3]);
      ws.g2d[(size_t)r * 3 + 1] = make_float4(a[4], a[5], a[6], a[7]);
      ws.g2d[(size_t)r * 3 + 2] = make_float4(a[8], 0.0f, 0.0f, 0.0f);
    }
    uint64_t big = __ballot(r < nrec && cnt > kBig);
    while (big) {
      const int l = __ffsll((unsigned long long)big) - 1;
      big &= big - 1;
      const uint32_t bc = __shfl(cnt, l, kWave), bp = __shfl(p0, l, kWave);
      float v[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) v[k] = 0.0f;
      for (uint32_t k = lane; k < bc; k += kWave) add_partial(ws.partials + (size_t)(bp + k) * 9, v);
      const float sum = wave_sum9_packed(v);
      float *dst = reinterpret_cast<float *>(ws.g2d + (size_t)(wbase + l) * 3);
      if (mine >= 0) dst[mine] = sum;
      if (mine == 8) dst[9] = dst[10] = dst[11] = 0.0f;
    }
  }
}

void launch_raster_bwd(const ViewInfo *views, const Ws &ws, const Sizes &sz, const float *t_final,
                       const uint32_t *last_pos, const float *dL_dimage, hipStream_t st) {
  if (sz.t_tot == 0) return;
#define BWD_ARGS views, ws, sz, t_final, last_pos, dL_dimage
  if (sz.ts == 16 && sz.t_tot <= kFewTiles && (sz.long_list == kLongAuto || sz.long_list == 0u)) {
    if (sz.persistent) launch_items<true, k_raster_bwd<16, true>>(sz.t_tot, BwdItem<16>::NT, st, BWD_ARGS);
    else launch_items<false, k_raster_bwd<16, false>>(sz.t_tot, BwdItem<16>::NT, st, BWD_ARGS);
    return;
  }
  switch ((sz.ts << 1) | (sz.persistent ? 1 : 0)) {
    case 16: launch_items<false, k_raster_bwd<8, false>>(sz.t_tot, BwdItem<8>::NT, st, BWD_ARGS); break;
    case 17: launch_items<true, k_raster_bwd<8, true>>(sz.t_tot, BwdItem<8>::NT, st, BWD_ARGS); break;
    case 64: launch_items<false, k_raster_bwd<32, false>>(sz.t_tot, BwdItem<32>::NT, st, BWD_ARGS); break;
    case 65: launch_items<true, k_raster_bwd<32, true>>(sz.t_tot, BwdItem<32>::NT, st, BWD_ARGS); break;
    case 33: launch_items<true, k_raster_bwd16<true>>(sz.t_tot, 256, st, BWD_ARGS); break;
    default: launch_items<false, k_raster_bwd16<false>>(sz.t_tot, 256, st, BWD_ARGS); break;
  }
#undef BWD_ARGS
}

void launch_reduce_pairs(const Ws &ws, const Sizes &sz, int32_t *step, hipStream_t st) {
  const uint32_t blocks = std::min<uint32_t>((sz.cap_rec + 255) / 256, 4096u);
  k_reduce_pairs<<<std::max(blocks, 1u), 256, 0, st>>>(ws, step);
}

}  // namespace gsr
