// LoG-based insertion of new Gaussians (Sec. 3.2, "Redundancy-free Gaussian
// Sampling", Eqs. 4-6) over all views of the plan:
//   P(I) = min(|| LoG_sigma * I ||, 1) per pixel (norm over the channels),
//   P_a  = max(P(I) - P(I~), 0), a Gaussian is inserted where P_a > tau_a,
//   S    = d / (2 sqrt(P(I)) f) for the inserted pixel, d the distance from
//          the back-projected centre (z from the depth map) to the camera.
//
// k_log_prob: one workgroup per tile of 64 x 32 or 64 x 16 pixels of a view.
// For each of the two images and each channel a horizontal pass convolves the
// tile's rows and a halo of R = ceil(3 sigma) rows (border pixels replicated)
// with the 1D Gaussian g and its second derivative h, reading each item's
// window straight into registers and leaving the results in LDS; a vertical
// pass finishes L = (h x g + g x h) * I, each thread one or two rows of four
// columns.  Writes P(I), optionally P(I~), and a byte mask of the inserting
// pixels.
//   Bound by VALU issue (44M instructions on six 1600x900 views; a tap of the
// vertical pass is a product, a fused one and a sum, whose rounding the mask
// depends on).  There 88 us; with all three channels of a 64 x 16 tile in
// 34 KB of LDS, read a value at a time, 115, and on eight 1903x1057 views,
// whose rows are not 16-byte aligned, the whole insertion 193 us, with their
// windows read a value at a time 352.  Four rows per thread take 98 us (fewer
// waves per SIMD), 64-row tiles 97 to 101; the next window or channel loaded
// ahead 91 to 97.
// k_ins_count / k_ins_scan / k_ins_write: stream compaction of the mask in
// ascending pixel order (counts per 4096 pixels, one scan, then each
// workgroup writes its pixels in order) with the new Gaussians' scale and
// world centre.
#include "kernels.hpp"
#include "util.hpp"

namespace gsr {

namespace {

constexpr int kTW = 64, kTT = 256;
// Below this many tiles of 16 rows a thread takes one row of one, above two
// rows of one of 32, with less of a halo.  The whole insertion: one view of
// 640x360 26 and 31 us, four of 960x540 (2,040) 43 and 46, three of 1601x901
// (4,446) 72 and 71, six of 1600x900 110 and 104.
constexpr uint32_t kSmallTiles = 2560;
constexpr int kInsBlock = 4096;  // pixels per compaction workgroup (256 threads x 16)

// View of a tile (the same in all lanes of the wave) and the number of tiles
// before the view's: 64 views at a time, a lane each.
template <int kTH>
__device__ __forceinline__ int view_of_ins_tile(const ViewInfo *__restrict__ views, int n_views, int tile, int &base) {
  const int lane = lane_id();
  base = 0;
  for (int v0 = 0; v0 < n_views; v0 += kWave) {
    int nt = 0;
    if (v0 + lane < n_views)
      nt = ((views[v0 + lane].w + kTW - 1) / kTW) * ((views[v0 + lane].h + kTH - 1) / kTH);
    const int incl = wave_incl_scan(nt);
    const uint64_t past = __ballot(tile < base + incl);
    if (past) {
      const int l = __ffsll((unsigned long long)past) - 1;
      base += __builtin_amdgcn_readlane(incl - nt, l);
      return v0 + l;
    }
    base += __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  return -1;
}

// R is a template parameter so that the tap loops unroll and the taps are
// read at compile-time indices.
// R rows to each side; tiles of kTH rows, kRows of them per thread.
template <int R, int kTH, int kRows>
__global__ __launch_bounds__(kTT) __attribute__((amdgpu_waves_per_eu(6))) void k_log_prob(
    const ViewInfo *__restrict__ views, int n_views, const float *__restrict__ gt, const float *__restrict__ rd,
    LogTaps taps, float tau, float *__restrict__ p_gt, float *__restrict__ p_rd, uint8_t *__restrict__ mask) {
  int base;
  static_assert(kTW / 4 * kTH / kRows == kTT);
  const int v = view_of_ins_tile<kTH>(views, n_views, blockIdx.x, base);
  if (v < 0) return;
  const ViewInfo vi = views[v];
  const int W = vi.w, H = vi.h;
  const int txs = (W + kTW - 1) / kTW;
  const int t = blockIdx.x - base;
  const int x0 = (t % txs) * kTW, y0 = (t / txs) * kTH;
  constexpr int rows = kTH + 2 * R;
  constexpr int RA = (R + 3) / 4 * 4;  // the filter radius rounded up to whole float4s
  __shared__ float4 A[rows][kTW / 4], B[rows][kTW / 4];  // rows * g, rows * h of one channel
  const int xg = threadIdx.x & 15, yg = threadIdx.x >> 4, yb = yg * kRows;
  // A thread's items of the horizontal pass are group xg of the rows yg,
  // yg + kTT / 16, ...; where the tile's windows lie inside the image it reads
  // four values at a time.
  constexpr int kItems = (rows + kTT / 16 - 1) / (kTT / 16), kVec = (4 + 2 * RA) / 4;
  const float *srcs[2] = {gt + 3 * vi.pix_off, rd + 3 * vi.pix_off};
  const bool whole = x0 >= RA && x0 + kTW + RA <= W;
  auto row_of = [&](int img, int ch, int i) {
    const int gy = min(max(y0 + yg + i * (kTT / 16) - R, 0), H - 1);
    return srcs[img] + ((int64_t)ch * H + gy) * W;
  };
  auto horizontal = [&](int r, const float *in) {
    float a[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = b[j] = 0.0f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) {
        a[j] = fmaf(taps.g[k], in[j + k], a[j]);
        b[j] = fmaf(taps.h[k], in[j + k], b[j]);
      }
    }
    A[r][xg] = make_float4(a[0], a[1], a[2], a[3]);
    B[r][xg] = make_float4(b[0], b[1], b[2], b[3]);
  };
  float P[2][kRows][4];
#pragma unroll
  for (int img = 0; img < 2; ++img) {
    float L2[kRows][4];
#pragma unroll
    for (int j = 0; j < kRows; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) L2[j][i] = 0.0f;
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
      const int ch = c == 2 ? 2 : 1 - c;  // the norm's square is l1 l1 + l0 l0 + l2 l2
      if (whole) {
#pragma unroll 1
        for (int i = 0; i < kItems && yg + i * (kTT / 16) < rows; ++i) {
          const Loose4 *rv = reinterpret_cast<const Loose4 *>(row_of(img, ch, i) + x0 + xg * 4 - RA);
          float buf[4 * kVec];
#pragma unroll
          for (int k = 0; k < kVec; ++k) {
            const Loose4 q = rv[k];
            buf[4 * k] = q.x;
            buf[4 * k + 1] = q.y;
            buf[4 * k + 2] = q.z;
            buf[4 * k + 3] = q.w;
          }
          horizontal(yg + i * (kTT / 16), buf + RA - R);
        }
      } else {
#pragma unroll 1
        for (int i = 0; i < kItems && yg + i * (kTT / 16) < rows; ++i) {
          const float *row = row_of(img, ch, i);
          float in[4 + 2 * R];
#pragma unroll
          for (int q = 0; q < 4 + 2 * R; ++q) in[q] = row[min(max(x0 + xg * 4 + q - R, 0), W - 1)];
          horizontal(yg + i * (kTT / 16), in);
        }
      }
      __syncthreads();
      float l[kRows][4];
#pragma unroll
      for (int k = 0; k < 2 * R + kRows; ++k) {
        const float4 a4 = A[yb + k][xg], b4 = B[yb + k][xg];
        const float a[4] = {a4.x, a4.y, a4.z, a4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          const int kk = k - j;  // tap index of this row for output row yb + j
          if (kk >= 0 && kk <= 2 * R) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float t = fmaf(taps.g[kk], b[i], taps.h[kk] * a[i]);
              l[j][i] = kk == 0 ? t : l[j][i] + t;
            }
          }
        }
      }
#pragma unroll
      for (int j = 0; j < kRows; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) L2[j][i] = fmaf(l[j][i], l[j][i], L2[j][i]);
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) P[img][j][i] = fminf(sqrtf(L2[j][i]), 1.0f);
  }
  const int gx = x0 + xg * 4;
  if (gx >= W) return;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const int gy = y0 + yb + j;
    if (gy >= H) break;
    const int64_t pix = vi.pix_off + (int64_t)gy * W + gx;
    uint32_t m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) m[i] = fmaxf(P[0][j][i] - P[1][j][i], 0.0f) > tau ? 1u : 0u;
    float *const p0 = p_gt + pix, *const p1 = p_rd ? p_rd + pix : p0;
    if (gx + 4 <= W && ((reinterpret_cast<uintptr_t>(p0) | reinterpret_cast<uintptr_t>(p1)) & 15u) == 0 &&
        (reinterpret_cast<uintptr_t>(mask + pix) & 3u) == 0) {
      *reinterpret_cast<float4 *>(p_gt + pix) = make_float4(P[0][j][0], P[0][j][1], P[0][j][2], P[0][j][3]);
      if (p_rd) *reinterpret_cast<float4 *>(p_rd + pix) = make_float4(P[1][j][0], P[1][j][1], P[1][j][2], P[1][j][3]);
      *reinterpret_cast<uint32_t *>(mask + pix) = m[0] | m[1] << 8 | m[2] << 16 | m[3] << 24;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (gx + i >= W) break;
        p_gt[pix + i] = P[0][j][i];
        if (p_rd) p_rd[pix + i] = P[1][j][i];
        mask[pix + i] = (uint8_t)m[i];
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_ins_count(const uint8_t *__restrict__ mask, int64_t n_pix,
                                                   uint32_t *__restrict__ counts) {
  __shared__ uint32_t red[4];
  const int64_t p0 = (int64_t)blockIdx.x * kInsBlock + (int64_t)threadIdx.x * 16;
  uint32_t c = 0;
  if (p0 + 16 <= n_pix) {  // mask bytes are 0 or 1: the popcount of the 16 bytes is their sum
    const uint4 m = *reinterpret_cast<const uint4 *>(mask + p0);
    c = __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
  } else {
    for (int i = 0; i < 16; ++i) c += (p0 + i < n_pix) ? mask[p0 + i] : 0u;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Exclusive offsets of the blocks' counts and the total (one workgroup), for
// more than kSumBlocks blocks; up to there k_ins_write adds the counts of the
// blocks before its own itself: on six 1600x900 views (2,110 blocks) 0.7 us
// there for a launch of 4.8.
constexpr uint32_t kSumBlocks = 4096;
__global__ __launch_bounds__(1024) void k_ins_scan(const uint32_t *__restrict__ counts, uint32_t nb,
                                                   uint32_t *__restrict__ offsets, uint32_t *__restrict__ total) {
  __shared__ uint32_t wsum[16];
  const uint32_t per = (nb + 1023) / 1024;
  const uint32_t b0 = threadIdx.x * per, b1 = min(b0 + per, nb);
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t s = 0;
  for (uint32_t b = b0; b < b1; ++b) s += counts[b];
  // inclusive scan of the threads' sums: within each wave by shuffles, then
  // over the 16 wave totals in the first wave
  uint32_t x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d);
    if (lane >= (uint32_t)d) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  if (w == 0) {
    uint32_t t = lane < 16 ? wsum[lane] : 0u;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const uint32_t y = __shfl_up(t, d);
      if (lane >= (uint32_t)d) t += y;
    }
    if (lane < 16) wsum[lane] = t;
  }
  __syncthreads();
  if (threadIdx.x == 1023) *total = wsum[15];
  uint32_t acc = x - s + (w > 0 ? wsum[w - 1] : 0u);
  for (uint32_t b = b0; b < b1; ++b) {
    offsets[b] = acc;
    acc += counts[b];
  }
}

template <bool SUM>
__global__ __launch_bounds__(256) void k_ins_write(const ViewInfo *__restrict__ views, int n_views,
                                                   const Cam *__restrict__ cams, const uint8_t *__restrict__ mask,
                                                   int64_t n_pix, const uint32_t *__restrict__ counts,
                                                   const uint32_t *__restrict__ offsets, uint32_t *__restrict__ total,
                                                   const float *__restrict__ p_gt, const float *__restrict__ depth,
                                                   uint32_t *__restrict__ out_pix, float *__restrict__ out_scale,
                                                   float *__restrict__ out_mean, int64_t capacity) {
  __shared__ uint32_t scan_tmp[4];
  constexpr int kPer = kInsBlock / 256;
  const int64_t p0 = (int64_t)blockIdx.x * kInsBlock + (int64_t)threadIdx.x * kPer;
  uint32_t bits = 0;
  if (p0 + kPer <= n_pix) {
    const uint4 m = *reinterpret_cast<const uint4 *>(mask + p0);
    const uint32_t w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
    for (int i = 0; i < kPer; ++i) bits |= ((w[i >> 2] >> (8 * (i & 3))) & 1u) << i;
  } else {
    for (int i = 0; i < kPer; ++i)
      if (p0 + i < n_pix && mask[p0 + i]) bits |= 1u << i;
  }
  const uint32_t mine = __popc(bits);
  uint32_t block_total;
  const uint32_t before = block_excl_scan<256>(mine, scan_tmp, block_total);
  uint32_t first;
  if (SUM) {
    uint32_t s = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 256) s += counts[b];
    __syncthreads();
    (void)block_excl_scan<256>(s, scan_tmp, first);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = first + block_total;
  } else {
    first = offsets[blockIdx.x];
  }
  uint32_t k = first + before;
  if (bits == 0) return;
  // view of the thread's first pixel (binary search), then forward at the
  // (rare) view boundary inside its 16 pixels
  int v = 0;
  for (int hi = n_views - 1; v < hi;) {
    const int mid = (v + hi + 1) >> 1;
    if ((int64_t)views[mid].pix_off <= p0) v = mid;
    else hi = mid - 1;
  }
  int64_t next = v + 1 < n_views ? (int64_t)views[v + 1].pix_off : INT64_MAX;
  ViewInfo vi = views[v];
  Cam c = cams[v];
  for (int i = 0; i < kPer; ++i) {
    if (!(bits >> i & 1u)) continue;
    const int64_t p = p0 + i;
    while (p >= next) {
      ++v;
      vi = views[v];
      c = cams[v];
      next = v + 1 < n_views ? (int64_t)views[v + 1].pix_off : INT64_MAX;
    }
    if ((int64_t)k < capacity) {
      const uint32_t local = (uint32_t)(p - vi.pix_off);  // a view's pixels fit 32 bits
      const int row = (int)(local / (uint32_t)vi.w), u = (int)(local - (uint32_t)row * (uint32_t)vi.w);
      const float z = depth[p];
      const float xc = z * (((float)u + 0.5f - c.cx) / c.fx);
      const float yc = z * (((float)row + 0.5f - c.cy) / c.fy);
      const float d = sqrtf(xc * xc + yc * yc + z * z);
      out_pix[k] = (uint32_t)p;
      out_scale[k] = d / (2.0f * sqrtf(p_gt[p]) * c.fx);
      // x_w = R^T (x_c - t)
      const float ex = xc - c.t[0], ey = yc - c.t[1], ez = z - c.t[2];
      out_mean[3 * k + 0] = c.R[0] * ex + c.R[3] * ey + c.R[6] * ez;
      out_mean[3 * k + 1] = c.R[1] * ex + c.R[4] * ey + c.R[7] * ez;
      out_mean[3 * k + 2] = c.R[2] * ex + c.R[5] * ey + c.R[8] * ez;
    }
    ++k;
  }
}

}  // namespace

uint32_t ins_tiles(const ViewInfo *views_host, int n_views, bool &small) {
  auto tiles = [&](int th) {
    uint32_t n = 0;
    for (int v = 0; v < n_views; ++v)
      n += (uint32_t)(((views_host[v].w + kTW - 1) / kTW) * ((views_host[v].h + th - 1) / th));
    return n;
  };
  const uint32_t n = tiles(16);
  small = n < kSmallTiles;
  return small ? n : tiles(32);
}

uint32_t ins_blocks(int64_t n_pix) { return (uint32_t)((n_pix + kInsBlock - 1) / kInsBlock); }

void launch_log_insert(const ViewInfo *views_d, int n_views, uint32_t n_tiles, bool small, int64_t n_pix, const Cam *cams,
                       const float *gt, const float *rd, const float *depth, const LogTaps &taps, float tau,
                       float *p_gt, float *p_rd, uint8_t *mask, uint32_t *counts, uint32_t *offsets,
                       uint32_t *total, uint32_t *out_pix, float *out_scale, float *out_mean, int64_t capacity,
                       hipStream_t st) {
  if (n_tiles == 0) return;
#define GSR_LOG_PROB(RR)                                                                                          \
  case RR:                                                                                                        \
    if (small)                                                                                                    \
      k_log_prob<RR, 16, 1><<<n_tiles, kTT, 0, st>>>(views_d, n_views, gt, rd, taps, tau, p_gt, p_rd, mask);       \
    else                                                                                                          \
      k_log_prob<RR, 32, 2><<<n_tiles, kTT, 0, st>>>(views_d, n_views, gt, rd, taps, tau, p_gt, p_rd, mask);       \
    break;
  switch (taps.R) {
    GSR_LOG_PROB(1)
    GSR_LOG_PROB(2)
    GSR_LOG_PROB(3)
    GSR_LOG_PROB(4)
    default: GSR_LOG_PROB(5)
  }
#undef GSR_LOG_PROB
  const uint32_t nb = ins_blocks(n_pix);
  k_ins_count<<<nb, 256, 0, st>>>(mask, n_pix, counts);
  if (nb <= kSumBlocks) {
    k_ins_write<true><<<nb, 256, 0, st>>>(views_d, n_views, cams, mask, n_pix, counts, offsets, total, p_gt, depth,
                                          out_pix, out_scale, out_mean, capacity);
    return;
  }
  k_ins_scan<<<1, 1024, 0, st>>>(counts, nb, offsets, total);
  k_ins_write<false><<<nb, 256, 0, st>>>(views_d, n_views, cams, mask, n_pix, counts, offsets, total, p_gt, depth,
                                         out_pix, out_scale, out_mean, capacity);
}

}  // namespace gsr
