// Depth sort and tile binning, as stable counting (LSD radix) passes on
// 8- to 11-bit digits -- no global atomics on contended addresses:
//
//  sort      the visible records by their depth bits (four passes; stable,
//            so equal depths keep record order, which is Gaussian order
//            within a view);
//  emission  every (record, tile) pair in depth-sorted record order: the
//            global tile id as key, the record as value, at the record's
//            pair offset (a scan of the rectangle areas in that order);
//  tile sort the pairs by tile id (one pass up to 2^11 tiles, two up to
//            2^20): being stable, it
//            leaves each tile's list in (depth, record) order, the
//            compositing order, so no per-tile sort is needed -- together
//            the passes sort the 64-bit (tile | depth) keys;
//  ranges    list start and length of every tile from the sorted ids, and
//            its longest-first key (an 8-bit length code);
//  order     the longest-first tile order, one counting pass over the codes.
//
// A pass is a per-block digit histogram, a scan of each digit's counts over
// the blocks, and a scatter that scans the digits' totals itself, ranks each
// block's items by digit with wave ballots and writes them through LDS in
// digit runs; small inputs are sorted in LDS runs and merged.  Far-away
// Gaussians crowd into the few tiles around the vanishing point of a street
// scene; per-pair atomic slot claims on those tiles would serialise, the
// counting passes do not.
#include <algorithm>

#include "kernels.hpp"
#include "util.hpp"

namespace gsr {

constexpr int kRdxNT = 512;  // threads per counting-pass block
// items per lane: 4 (2048 per block) for inputs below kRdxBig items, so a
// pass spreads over enough workgroups, else 16 (8192 per block).  A block's
// rounds are a chain, so eight waves rank a chunk faster than four.
constexpr int kRdxIPL = 4, kRdxBigIPL = 16;
constexpr uint32_t kRdxBig = 1u << 23;
constexpr int kScanNT = 256, kScanIPT = 16;
constexpr uint32_t kScanChunk = kScanNT * kScanIPT;

// Longest-first code of a list length: 16 steps per octave (the exponent
// and top four mantissa bits of the length as a float), inverted, so the
// longest lists come first; lengths from 2^16 up share the first code.
__device__ __forceinline__ uint32_t length_key(uint32_t n) {
  if (n == 0) return 255u;
  const uint32_t code = (__float_as_uint((float)n) >> 19) - (127u << 4);  // 0 for n = 1
  return 255u - min(code, 255u);
}

__device__ __forceinline__ uint32_t n_items(const uint32_t *count_dev, uint32_t cap) {
  return count_dev ? min(*count_dev, cap) : cap;
}

// Emission: each wave takes 64 consecutive records of the depth order (their
// indices perm[i] and tile records srect[i] are read in order); their pairs
// form one contiguous range (offs[i] is the first pair of sorted record i).
// A record of at most kEmitSmall pairs is written by its own lane, stepping
// through its tile rectangle; the lanes' stores fall into that one range.
// Bigger footprints are written by the whole wave, 64 pairs per step.
constexpr uint32_t kEmitSmall = 8;

__global__ __launch_bounds__(256) void k_emit(Ws ws, Sizes sz,
                                              const uint32_t *__restrict__ perm, const uint4 *__restrict__ srect,
                                              const uint32_t *__restrict__ offs,
                                              uint32_t *__restrict__ keys, uint32_t *__restrict__ vals) {
  if (ws.scalars[kOverflow]) return;
  const uint32_t nrec = ws.scalars[kNumRecords];
  const int lane = lane_id();
  const uint32_t wave_stride = gridDim.x * (blockDim.x / kWave) * kWave;
  for (uint32_t wbase = (blockIdx.x * (blockDim.x / kWave) + wave_id()) * kWave; wbase < nrec;
       wbase += wave_stride) {
    const uint32_t i = wbase + lane;
    uint32_t tx0 = 0, tx1 = 0, ty0 = 0, w = 1, cnt = 0, off = 0, rec = 0, tbase = 0, tpitch = 0;
    if (i < nrec) {
      rec = perm[i];
      const uint4 rc = srect[i];  // rectangle, first tile, row pitch
      tx0 = rc.x & 0xFFFFu;
      tx1 = rc.x >> 16;
      ty0 = rc.y & 0xFFFFu;
      w = tx1 - tx0 + 1;
      cnt = w * ((rc.y >> 16) - ty0 + 1);
      tbase = rc.z - ty0 * rc.w - tx0;  // so that tbase + ty * pitch + tx is the tile's id
      tpitch = rc.w;
      off = offs[i];
      const uint32_t last = rc.z + ((rc.y >> 16) - ty0) * rc.w + (tx1 - tx0);
      // inconsistent pair offsets, or a tile that the plan has not (the sort
      // takes the bits that the tiles need, so nothing behind it would see one)
      if (off + cnt > sz.cap_pairs || max(rc.z, last) >= sz.t_tot) {
        ws.scalars[kOverflow] = 3u;
        cnt = 0;
      }
    }
    if (cnt <= kEmitSmall) {
      uint32_t tx = tx0, row = tbase + ty0 * tpitch;
      for (uint32_t k = 0; k < cnt; ++k) {
        keys[off + k] = row + tx;
        vals[off + k] = rec;
        if (++tx > tx1) {
          tx = tx0;
          row += tpitch;
        }
      }
    }
    uint64_t big = __ballot(cnt > kEmitSmall);
    while (big) {
      const int l = __ffsll((unsigned long long)big) - 1;
      big &= big - 1;
      const uint32_t b_cnt = __shfl(cnt, l, kWave), b_off = __shfl(off, l, kWave), b_rec = __shfl(rec, l, kWave);
      const uint32_t b_tx0 = __shfl(tx0, l, kWave), b_w = __shfl(w, l, kWave);
      const uint32_t b_row0 = __shfl(tbase + ty0 * tpitch, l, kWave), b_pitch = __shfl(tpitch, l, kWave);
      for (uint32_t k = lane; k < b_cnt; k += kWave) {
        const uint32_t r = k / b_w, c = k - r * b_w;
        keys[b_off + k] = b_row0 + r * b_pitch + b_tx0 + c;
        vals[b_off + k] = b_rec;
      }
    }
  }
}

// Chunk of a counting-pass workgroup, given the number of chunks holding
// live items.  Workgroups go to the 8 XCDs in turn, so the live chunks are
// dealt out as 8 contiguous ranges, one per XCD: neighbouring chunks then
// share the cache lines of their digit-major histogram entries, and of their
// short digit runs in the output, in one XCD's L2 instead of writing parts
// of the same lines from different XCDs.  Chunks past the live ones keep
// their workgroup's index.
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t live_chunks) {
  const uint32_t b = blockIdx.x;
  if (b >= live_chunks) return b;
  const uint32_t x = b & 7u, q = live_chunks >> 3, r = live_chunks & 7u;
  return x * q + min(x, r) + (b >> 3);
}

// Lanes of the wave whose BITS-bit digit equals this lane's, among `live`:
// one ballot per bit; a lane differs from this one where the ballot of some
// bit differs from this lane's own bit (spread over a word as 0 or ~0), and
// those differences are OR-ed up per 32-lane half.
template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool live) {
  uint32_t lo = 0u, hi = 0u;
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const uint32_t x = (uint32_t)((int32_t)(d << (31 - b)) >> 31);
    const uint64_t m = __ballot(x != 0u);
    lo |= (uint32_t)m ^ x;
    hi |= (uint32_t)(m >> 32) ^ x;
  }
  return ((uint64_t)~hi << 32 | (uint64_t)~lo) & __ballot(live);
}

// 2a. Digit histogram of one block's chunk (IPL items per lane) for digits
// of BITS bits (2^BITS bins), stored digit-major in rows of `pitch` chunks:
// hist[d * pitch + chunk].  Chunks past the live items are neither written
// nor read.  Each wave loads its items first, then counts
// them 64 at a time: one LDS atomic when all 64 share a digit (as the high
// depth bits mostly do), else one per lane.
template <int IPL, int BITS>
__global__ __launch_bounds__(kRdxNT) void k_digit_hist(const uint32_t *__restrict__ scalars,
                                                       const uint32_t *__restrict__ keys,
                                                       const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                       int shift, uint32_t pitch, uint32_t *__restrict__ hist) {
  constexpr uint32_t CHUNK = kRdxNT * IPL;
  constexpr uint32_t RADIX = 1u << BITS, MASK = RADIX - 1u;
  __shared__ uint32_t h[RADIX];
  if (scalars[kOverflow]) return;
  const uint32_t t = threadIdx.x;
  const uint32_t n = n_items(count_dev, cap);
  const uint32_t live_chunks = n / CHUNK + (n % CHUNK != 0u);
  if (blockIdx.x >= live_chunks) return;  // uniform
  const uint32_t c = xcd_chunk(live_chunks);
  for (uint32_t d = t; d < RADIX; d += kRdxNT) h[d] = 0u;
  __syncthreads();
  {
    const uint32_t lo = c * CHUNK + (uint32_t)wave_id() * (CHUNK / (kRdxNT / kWave)) + (uint32_t)lane_id();
    uint32_t d[IPL];
#pragma unroll
    for (int r = 0; r < IPL; ++r) {
      const uint32_t i = lo + (uint32_t)r * kWave;
      d[r] = i < n ? (keys[i] >> shift) & MASK : 0u;
    }
#pragma unroll
    for (int r = 0; r < IPL; ++r) {
      const bool live = lo + (uint32_t)r * kWave < n;  // lane 0 is live if any lane is
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d[r]);
      const uint64_t all = __ballot(live);
      if (__ballot(live && d[r] == d0) == all) {
        if (lane_id() == 0 && all) atomicAdd(&h[d0], (uint32_t)__popcll(all));
      } else if (live) {
        atomicAdd(&h[d[r]], 1u);
      }
    }
  }
  __syncthreads();
  for (uint32_t d = t; d < RADIX; d += kRdxNT) hist[d * pitch + c] = h[d];
}

// 2b. Each digit's row of chunk counts turned into its exclusive prefix sums,
// and the row totals, in one launch: a row per workgroup (WG), or with few
// chunks a row per wave.  The scatter's blocks scan the 2^BITS totals
// themselves, so no device-wide scan over all rows (two launches, or one slow
// workgroup) is needed.
template <bool WG>
__global__ __launch_bounds__(256) void k_digit_rows(const uint32_t *__restrict__ scalars,
                                                    const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                    uint32_t chunk, uint32_t pitch, uint32_t *__restrict__ hist,
                                                    uint32_t *__restrict__ totals) {
  __shared__ uint32_t red[4];
  if (scalars[kOverflow]) return;
  const uint32_t n = n_items(count_dev, cap);
  const uint32_t live = n / chunk + (n % chunk != 0u);
  const uint32_t d = WG ? blockIdx.x : blockIdx.x * 4u + (uint32_t)wave_id();
  const uint32_t t = WG ? threadIdx.x : (uint32_t)lane_id();
  constexpr uint32_t STEP = (WG ? 256u : 64u) * 4u;
  uint4 *row = reinterpret_cast<uint4 *>(hist + (size_t)d * pitch);  // pitch is a multiple of 4
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < live; b0 += STEP) {
    const uint32_t i = b0 + 4u * t;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (i < live) {
      x = row[i / 4];
      if (i + 1 >= live) x.y = 0u;  // the row's last word group may hold stale words
      if (i + 2 >= live) x.z = 0u;
      if (i + 3 >= live) x.w = 0u;
    }
    const uint32_t mine = (x.x + x.y) + (x.z + x.w);
    uint32_t before, total;
    if (WG) {
      before = block_excl_scan<256>(mine, red, total);
    } else {
      const uint32_t incl = wave_incl_scan(mine);
      before = incl - mine;
      total = (uint32_t)__shfl(incl, kWave - 1, kWave);
    }
    before += carry;
    if (i < live) row[i / 4] = make_uint4(before, before + x.x, before + x.x + x.y, before + x.x + x.y + x.z);
    carry += total;
  }
  if (t == 0) totals[d] = carry;
}

// Device-wide exclusive scan of data[0, len), len = min(*count_dev, cap) (cap
// if NULL): chunk sums, then each chunk
// scanned with its offset, the sum of the totals before it (added up by the
// chunk's own workgroup, or over many chunks by a single-block scan).  Global
// accesses are coalesced; the per-thread runs of 16 words are read from LDS
// with a skew of one word per 16, so the 64 lanes hit distinct banks.
__device__ __forceinline__ uint32_t skew(uint32_t j) { return j + (j >> 4); }

__global__ __launch_bounds__(kScanNT) void k_scan_reduce(const uint32_t *__restrict__ data,
                                                         const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                         uint32_t *__restrict__ part) {
  __shared__ uint32_t s[kScanNT / kWave];
  const uint32_t len = n_items(count_dev, cap);
  const uint32_t lo = blockIdx.x * kScanChunk;
  if (lo >= len) {  // uniform
    if (threadIdx.x == 0) part[blockIdx.x] = 0u;
    return;
  }
  uint32_t acc = 0;
#pragma unroll
  for (int i = 0; i < kScanIPT; ++i) {
    const uint32_t j = lo + (uint32_t)i * kScanNT + threadIdx.x;
    acc += j < len ? data[j] : 0u;
  }
  uint32_t total;
  block_excl_scan<kScanNT>(acc, s, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_top(uint32_t *__restrict__ part, uint32_t nb) {
  __shared__ uint32_t s[1024 / kWave];
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < nb; b0 += 1024) {
    const uint32_t i = b0 + threadIdx.x;
    const uint32_t x = i < nb ? part[i] : 0u;
    uint32_t total;
    const uint32_t e = block_excl_scan<1024>(x, s, total);
    if (i < nb) part[i] = carry + e;
    carry += total;
  }
}

// Exclusive scan of NT*16 words at data + lo (words past len read as 0 and
// are not written), plus `carry`; returns the chunk total.
template <int NT>
__device__ __forceinline__ uint32_t scan_chunk(uint32_t *__restrict__ data, uint32_t lo, uint32_t len,
                                               uint32_t carry, uint32_t *lds, uint32_t *red) {
  constexpr uint32_t C = NT * 16;
  const uint32_t t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t j = (uint32_t)i * NT + t;
    lds[skew(j)] = lo + j < len ? data[lo + j] : 0u;
  }
  __syncthreads();
  uint32_t x[16], acc = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    x[i] = lds[skew(t * 16 + i)];
    acc += x[i];
  }
  uint32_t total;
  uint32_t run = carry + block_excl_scan<NT>(acc, red, total);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    lds[skew(t * 16 + i)] = run;
    run += x[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t j = (uint32_t)i * NT + t;
    if (lo + j < len) data[lo + j] = lds[skew(j)];
  }
  __syncthreads();
  (void)C;
  return total;
}

// Small scans in one workgroup of 1024 threads, 16K words per step.
__global__ __launch_bounds__(1024) void k_scan_one(uint32_t *__restrict__ data, const uint32_t *__restrict__ count_dev,
                                                   uint32_t cap) {
  const uint32_t len = n_items(count_dev, cap);
  __shared__ uint32_t lds[1024 * 16 + 1024];
  __shared__ uint32_t red[1024 / kWave];
  uint32_t carry = 0;
  for (uint32_t base = 0; base < len; base += 1024u * 16u) carry += scan_chunk<1024>(data, base, len, carry, lds, red);
}

// SUM_BEFORE: part holds the chunk totals, and each workgroup adds up those
// before its chunk itself (at most kScanFusedMax words, read from L2), which
// saves the launch of the single-block scan of the totals.  Otherwise part
// holds the chunks' offsets.
template <bool SUM_BEFORE>
__global__ __launch_bounds__(kScanNT) void k_scan_down(uint32_t *__restrict__ data,
                                                       const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                       const uint32_t *__restrict__ part) {
  __shared__ uint32_t lds[kScanChunk + kScanChunk / 16];
  __shared__ uint32_t red[kScanNT / kWave];
  const uint32_t len = n_items(count_dev, cap);
  if (blockIdx.x * kScanChunk >= len) return;  // uniform
  uint32_t carry;
  if (SUM_BEFORE) {
    uint32_t c = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanNT) c += part[i];
    block_excl_scan<kScanNT>(c, red, carry);
  } else {
    carry = part[blockIdx.x];
  }
  scan_chunk<kScanNT>(data, blockIdx.x * kScanChunk, len, carry, lds, red);
}

// 2c. Stable scatter of one block's chunk by digit, from the row prefixes and
// totals of its digits.  Wave w owns the w-th
// eighth of the chunk and loads all of it first (IPL items per lane).  It
// ranks its items by digit round by round (64 items, in order) with ballot
// matches and its own running digit counts in LDS, so no workgroup barrier
// is needed per round.  The block then places its items in LDS in local
// digit order (stable: waves and rounds in item order) and writes each
// digit's run to its global offset, contiguously.  vals_in = NULL: the
// values are the item indices.  With area_out, the values are records, and
// their tile-rectangle areas and tile records (rect_out) are written beside
// them.
// Counts within a block fit 16 bits, so two blocks of 8192 items and 9-bit
// digits share a CU's 160 KB of LDS (with 32-bit counts one did, and a pass
// over 67M pairs took 342 us).
template <int IPL, int BITS>
struct ScatterLds {
  uint32_t key[kRdxNT * IPL];
  uint32_t val[kRdxNT * IPL];
  uint16_t wcnt[kRdxNT / kWave][1u << BITS];  // running, then starting, counts per wave and digit
  uint32_t gdiff[1u << BITS];                 // global start of each digit for this block, less its local start
  uint32_t scan[kRdxNT / kWave];
};

template <int IPL, int BITS>
__global__ __launch_bounds__(kRdxNT) void k_digit_scatter(const uint32_t *__restrict__ scalars,
                                                          const uint32_t *__restrict__ keys_in,
                                                          const uint32_t *__restrict__ vals_in,
                                                          uint32_t *__restrict__ keys_out,
                                                          uint32_t *__restrict__ vals_out,
                                                          const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                          int shift, uint32_t pitch,
                                                          const uint32_t *__restrict__ hist,
                                                          const uint32_t *__restrict__ totals,
                                                          const uint4 *__restrict__ rect,
                                                          uint32_t *__restrict__ area_out,
                                                          uint4 *__restrict__ rect_out) {
  constexpr int NW = kRdxNT / kWave;
  constexpr uint32_t CHUNK = kRdxNT * IPL;
  constexpr uint32_t RADIX = 1u << BITS, MASK = RADIX - 1u;
  constexpr int DPT = RADIX > kRdxNT ? (int)(RADIX / kRdxNT) : 1;  // digits per thread, consecutive: t * DPT + k
  __shared__ ScatterLds<IPL, BITS> S;
  if (scalars[kOverflow]) return;
  const uint32_t t = threadIdx.x;
  const int w = wave_id(), lane = lane_id();
  const uint32_t n = n_items(count_dev, cap);
  const uint32_t c = xcd_chunk(n / CHUNK + (n % CHUNK != 0u)), blo = c * CHUNK;
  if (blo >= n) return;  // uniform: nothing of this block is live
  const uint32_t m = min(CHUNK, n - blo);
  uint32_t dtot[DPT], drow[DPT];
#pragma unroll
  for (int e = 0; e < DPT; ++e) {
    const uint32_t d = t * DPT + (uint32_t)e;
    const bool in = d < RADIX;
    if (in)
#pragma unroll
      for (int k = 0; k < NW; ++k) S.wcnt[k][d] = 0u;
    dtot[e] = in ? totals[d] : 0u;
    drow[e] = in ? hist[d * pitch + c] : 0u;
  }
  const uint32_t lo = blo + (uint32_t)w * (CHUNK / NW);
  uint32_t key[IPL], val[IPL], rk[IPL];
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const uint32_t i = lo + (uint32_t)r * kWave + (uint32_t)lane;
    key[r] = i < n ? keys_in[i] : 0u;
    val[r] = i < n ? (vals_in ? vals_in[i] : i) : 0u;
  }
  {
    // global start of each digit (a scan of the totals) and of this block in it
    uint32_t sum = 0, total;
#pragma unroll
    for (int e = 0; e < DPT; ++e) sum += dtot[e];
    uint32_t run = block_excl_scan<kRdxNT>(sum, S.scan, total);
#pragma unroll
    for (int e = 0; e < DPT; ++e) {
      if (t * DPT + (uint32_t)e < RADIX) S.gdiff[t * DPT + (uint32_t)e] = run + drow[e];
      run += dtot[e];
    }
  }
  __syncthreads();
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const uint32_t i = lo + (uint32_t)r * kWave + (uint32_t)lane;
    const bool live = i < n;
    const uint32_t d = (key[r] >> shift) & MASK;
    const uint64_t eq = match_digit<BITS>(d, live);
    const uint32_t before = (uint32_t)__popcll(eq & lt);
    const uint32_t prior = S.wcnt[w][d];
    rk[r] = prior + before;
    if (live && before == 0) S.wcnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(eq));
  }
  __syncthreads();
  {
    // the thread's DPT consecutive digits: local starts in digit order, then
    // per digit in wave order
    uint32_t cnt[DPT][NW], tot = 0;
#pragma unroll
    for (int e = 0; e < DPT; ++e)
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        cnt[e][k] = t * DPT + (uint32_t)e < RADIX ? S.wcnt[k][t * DPT + (uint32_t)e] : 0u;
        tot += cnt[e][k];
      }
    uint32_t total;
    uint32_t run = block_excl_scan<kRdxNT>(tot, S.scan, total);
#pragma unroll
    for (int e = 0; e < DPT; ++e) {
      const uint32_t d = t * DPT + (uint32_t)e;
      if (d >= RADIX) break;
      S.gdiff[d] -= run;  // the thread's own entry
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        S.wcnt[k][d] = (uint16_t)run;
        run += cnt[e][k];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < IPL; ++r) {
    const uint32_t i = lo + (uint32_t)r * kWave + (uint32_t)lane;
    if (i < n) {
      const uint32_t p = S.wcnt[w][(key[r] >> shift) & MASK] + rk[r];
      S.key[p] = key[r];
      S.val[p] = val[r];
    }
  }
  __syncthreads();
  for (uint32_t j = t; j < m; j += kRdxNT) {
    const uint32_t k = S.key[j], v = S.val[j];
    const uint32_t d = (k >> shift) & MASK;
    const uint32_t g = S.gdiff[d] + j;
    if (g < cap) {
      keys_out[g] = k;
      vals_out[g] = v;
      if (area_out) {  // tile record and tile-rectangle area of record v
        const uint4 rc = rect[v];
        area_out[g] = ((rc.x >> 16) - (rc.x & 0xFFFFu) + 1) * ((rc.y >> 16) - (rc.y & 0xFFFFu) + 1);
        rect_out[g] = rc;
      }
    }
  }
}

// Small inputs (at most kMergeMax items, on the host's capacity) are sorted
// in two launches instead of three per digit: each workgroup sorts a run of
// kRunItems items in LDS (all digits), then every item finds its place by
// searching the other runs.  The searches grow with the square of the item
// count, so larger inputs take the passes.  A whole forward with either, the
// live items being less than the capacity of 65,536 (1920x1080): the depth sort
// (four passes) of 4,000 records 100 us and 123, of 25,000 110 and 133, of
// 65,000 124 and 139; the tile sort where it would take two passes (8,160 tiles)
// of 4,600 pairs 94 and 98, of 33,000 113 and 109, of 64,000 126 and 121, and
// where it would take one (1,450 tiles) 80 and 79, 90 and 88, 110 and 99.  So
// the line is the depth sort's; the tile sort, which would rather end at 30,000
// pairs or none, loses less there than the depth sort gains.
constexpr int kRunNT = 1024, kRunIPL = 4;
constexpr uint32_t kRunItems = kRunNT * kRunIPL;
constexpr uint32_t kMergeMax = 16 * kRunItems;

// Stable LDS sort of run blockIdx.x by the low 8 * n_digits bits of the keys.
// Wave w holds items [w * 256, +256) of the run's current order, 64 per round;
// a digit is ranked as in the scatter.  Items past the live ones sort last:
// they take the digit 255 and stand behind the live ones from the start.
// final_out: the only run, which writes the sorted records' areas and tile
// records too.
__global__ __launch_bounds__(kRunNT) void k_sort_runs(const uint32_t *__restrict__ scalars, const uint32_t *keys_in,
                                                      const uint32_t *vals_in, uint32_t *keys_out, uint32_t *vals_out,
                                                      const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                      int n_digits, const uint4 *__restrict__ rect,
                                                      uint32_t *__restrict__ area_out, uint4 *__restrict__ rect_out) {
  constexpr int NW = kRunNT / kWave;
  __shared__ uint32_t s_key[kRunItems], s_val[kRunItems], wcnt[NW][256], red[4];
  if (scalars[kOverflow]) return;
  const uint32_t n = n_items(count_dev, cap), lo = blockIdx.x * kRunItems;
  if (lo >= n) return;  // uniform
  const uint32_t m = min(kRunItems, n - lo);
  const uint32_t t = threadIdx.x;
  const int w = wave_id(), lane = lane_id();
  uint32_t key[kRunIPL], val[kRunIPL], rk[kRunIPL];
#pragma unroll
  for (int r = 0; r < kRunIPL; ++r) {
    const uint32_t i = (uint32_t)w * (kRunItems / NW) + (uint32_t)r * kWave + (uint32_t)lane;
    key[r] = i < m ? keys_in[lo + i] : 0xFFFFFFFFu;
    val[r] = i < m ? (vals_in ? vals_in[lo + i] : lo + i) : 0u;
  }
  for (int p = 0; p < n_digits; ++p) {
    const int shift = 8 * p;
#pragma unroll
    for (int k = 0; k < NW * 256 / kRunNT; ++k) wcnt[0][t + (uint32_t)k * kRunNT] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunIPL; ++r) {
      const uint32_t d = (key[r] >> shift) & 255u;
      const uint64_t eq = match_digit<8>(d, true);
      const uint32_t before = (uint32_t)__popcll(eq & lanemask_lt());
      const uint32_t prior = wcnt[w][d];
      rk[r] = prior + before;
      if (before == 0) wcnt[w][d] = prior + (uint32_t)__popcll(eq);
    }
    __syncthreads();
    uint32_t tot = 0, incl = 0;
    if (t < 256) {
#pragma unroll
      for (int k = 0; k < NW; ++k) tot += wcnt[k][t];
      incl = wave_incl_scan(tot);
      if (lane == kWave - 1) red[w] = incl;
    }
    __syncthreads();
    if (t < 256) {
      uint32_t run = incl - tot;
      for (int k = 0; k < w; ++k) run += red[k];
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t c = wcnt[k][t];
        wcnt[k][t] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunIPL; ++r) {
      const uint32_t at = wcnt[w][(key[r] >> shift) & 255u] + rk[r];
      s_key[at] = key[r];
      s_val[at] = val[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunIPL; ++r) {
      const uint32_t i = (uint32_t)w * (kRunItems / NW) + (uint32_t)r * kWave + (uint32_t)lane;
      key[r] = s_key[i];
      val[r] = s_val[i];
    }
  }
#pragma unroll
  for (int r = 0; r < kRunIPL; ++r) {
    const uint32_t i = (uint32_t)w * (kRunItems / NW) + (uint32_t)r * kWave + (uint32_t)lane;
    if (i < m) {
      keys_out[lo + i] = key[r];
      vals_out[lo + i] = val[r];
      if (area_out) {
        const uint4 rc = rect[val[r]];
        area_out[lo + i] = ((rc.x >> 16) - (rc.x & 0xFFFFu) + 1) * ((rc.y >> 16) - (rc.y & 0xFFFFu) + 1);
        rect_out[lo + i] = rc;
      }
    }
  }
}

// Place of every item of the sorted runs in the whole: its index in its run,
// plus the items of the other runs that come before it (equal keys of earlier
// runs count, of later runs not, so the sort is stable).  Eight runs are
// searched at a time, so their dependent loads overlap.
__global__ __launch_bounds__(256) void k_merge_runs(const uint32_t *__restrict__ scalars,
                                                    const uint32_t *__restrict__ keys_in,
                                                    const uint32_t *__restrict__ vals_in,
                                                    uint32_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out,
                                                    const uint32_t *__restrict__ count_dev, uint32_t cap,
                                                    const uint4 *__restrict__ rect,
                                                    uint32_t *__restrict__ area_out, uint4 *__restrict__ rect_out) {
  if (scalars[kOverflow]) return;
  const uint32_t n = n_items(count_dev, cap);
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const uint32_t x = keys_in[i], val = vals_in[i];
  const uint32_t own = i / kRunItems, runs = n / kRunItems + (n % kRunItems != 0u);
  uint32_t at = i - own * kRunItems;
  for (uint32_t g = 0; g < runs; g += 8) {
    uint32_t pos[8], len[8];
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      const uint32_t r = g + q;
      pos[q] = 0u;
      len[q] = r < runs && r != own ? min(kRunItems, n - r * kRunItems) : 0u;
    }
#pragma unroll 1
    for (uint32_t step = kRunItems; step > 0; step >>= 1) {
      uint32_t v[8];
#pragma unroll
      for (uint32_t q = 0; q < 8; ++q) {
        const bool in = pos[q] + step <= len[q];
        v[q] = in ? keys_in[(g + q) * kRunItems + pos[q] + step - 1u] : 0xFFFFFFFFu;
      }
#pragma unroll
      for (uint32_t q = 0; q < 8; ++q) {
        const bool before = g + q < own ? v[q] <= x : v[q] < x;
        pos[q] += before && pos[q] + step <= len[q] ? step : 0u;
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) at += pos[q];
  }
  keys_out[at] = x;
  vals_out[at] = val;
  if (area_out) {
    const uint4 rc = rect[val];
    area_out[at] = ((rc.x >> 16) - (rc.x & 0xFFFFu) + 1) * ((rc.y >> 16) - (rc.y & 0xFFFFu) + 1);
    rect_out[at] = rc;
  }
}

// 3a. List bounds from the sorted tile ids: the first entry of a tile writes
// its start, the last one its end (into tile_count, turned into the length
// by k_tile_ranges).  Both arrays are zeroed by the forward beforehand.
// Each thread takes four consecutive ids with one 16-byte load.
__global__ void k_tile_bounds(Ws ws, Sizes sz, const uint32_t *__restrict__ tiles) {
  if (ws.scalars[kOverflow]) return;
  const uint32_t n = min(ws.scalars[kNumPairs], sz.cap_pairs);
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; 4 * q < n; q += stride) {
    const uint32_t i0 = 4 * q;
    uint32_t t[6];
    t[0] = i0 > 0 ? tiles[i0 - 1] : 0xFFFFFFFFu;
    if (i0 + 4 <= n) {
      const uint4 v = *reinterpret_cast<const uint4 *>(tiles + i0);  // i0 is a multiple of 4
      t[1] = v.x; t[2] = v.y; t[3] = v.z; t[4] = v.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) t[1 + k] = i0 + k < n ? tiles[i0 + k] : 0xFFFFFFFFu;
    }
    t[5] = i0 + 4 < n ? tiles[i0 + 4] : 0xFFFFFFFFu;
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
      const uint32_t i = i0 + (uint32_t)k - 1;
      if (i >= n) break;
      const uint32_t tl = t[k];
      if (tl >= sz.t_tot) {
        ws.scalars[kOverflow] = 3u;
        continue;
      }
      if (t[k - 1] != tl) ws.tile_start[tl] = i;
      if (t[k + 1] != tl) ws.tile_count[tl] = i + 1;
    }
  }
}

// 3b. Per tile the list bounds, the longest-first code and, per block of
// kOrderNT tiles, the code histogram (codes of 8 bits) and the number of
// long lists.  The bounds come from k_tile_bounds,
// or (SEARCH) from a binary search for each tile's first sorted entry: on 67M
// pairs the search takes 37 us and the pass over them 63, on 4.3M 17 and 10.
constexpr int kOrderNT = 1024;
// A list is long (the backward walks it with a wave per 8 x 8 block, see
// raster_bwd.hip) from a share of all pairs, where it would outlast the rest:
// one wave takes about five times as long per entry alone as it does among
// five others, so a list of a 5000th of all pairs takes as long as the 1024
// SIMDs do for everything.  Measured at shares of 2048, 4096, 8192 and 16384:
// four views of the rig 520, 520, 543 and 589 us, one 1080p view of 500k 158,
// 162, 176 and 181, four 800x450 views of 100k 107, 105, 105 and 106 (271
// without).  A fixed length does not carry over: from 512 and 1024 entries
// the whole rig takes 661 and 626 us (626 with the share), 40 mixed views 7.5
// ms from 1024 (6.5).  This is the rule of kLongAuto; every other long_list is
// the length that its caller wants.
constexpr uint32_t kLongShare = 4096, kLongMin = 32;

__device__ __forceinline__ uint32_t lower_bound(const uint32_t *__restrict__ a, uint32_t n, uint32_t x) {
  uint32_t lo = 0;
  while (n > 0) {
    const uint32_t half = n >> 1;
    const bool below = a[lo + half] < x;
    lo += below ? half + 1 : 0u;
    n = below ? n - half - 1 : half;
  }
  return lo;
}

template <bool SEARCH>
__global__ __launch_bounds__(kOrderNT) void k_tile_ranges(Ws ws, Sizes sz, const uint32_t *__restrict__ tiles,
                                                          uint32_t *__restrict__ codes,
                                                          uint32_t *__restrict__ code_hist) {
  __shared__ uint32_t start[SEARCH ? kOrderNT + 1 : 1], h[256];
  if (ws.scalars[kOverflow]) return;
  const uint32_t t = threadIdx.x, tile = blockIdx.x * kOrderNT + t;
  if (t < 256) h[t] = 0u;
  if (SEARCH) {
    const uint32_t n = min(ws.scalars[kNumPairs], sz.cap_pairs);
    start[t] = lower_bound(tiles, n, tile);
    if (t == 0) start[kOrderNT] = lower_bound(tiles, n, tile + kOrderNT);
  }
  __syncthreads();
  const bool valid = tile < sz.t_tot;
  uint32_t len = 0;
  if (valid) {
    if (SEARCH) {
      len = start[t + 1] - start[t];
      ws.tile_start[tile] = start[t];
    } else {
      const uint32_t end = ws.tile_count[tile];
      len = end ? end - ws.tile_start[tile] : 0u;
    }
    const uint32_t code = length_key(len);
    ws.tile_count[tile] = len;
    codes[tile] = code;
    atomicAdd(&h[code], 1u);
  }
  const uint32_t long_len = sz.long_list == kLongAuto ? max(kLongMin, ws.scalars[kNumPairs] / kLongShare) : sz.long_list;
  (void)wave_atomic_inc(ws.scalars + kNumLong, valid && len >= long_len);
  __syncthreads();
  if (t < 256) code_hist[(size_t)blockIdx.x * 256 + t] = h[t];
}

// 4. Longest-first tile order: a stable counting pass over the codes in one
// launch.  Each block adds up the code counts of all blocks and of those
// before it (nb rows of 256), scans the codes and ranks its tiles.
__global__ __launch_bounds__(kOrderNT) void k_tile_order(Ws ws, Sizes sz, const uint32_t *__restrict__ codes,
                                                         const uint32_t *__restrict__ code_hist) {
  constexpr int NW = kOrderNT / kWave;
  __shared__ uint32_t part[2][4][256], base[256], wcnt[NW][256], red[4];
  if (ws.scalars[kOverflow]) return;
  const uint32_t t = threadIdx.x, nb = gridDim.x;
  const int w = wave_id();
  {
    // thread (q, d): blocks q, q + 4, ... of code d
    const uint32_t d = t & 255u, q = t >> 8;
    uint32_t all = 0, before = 0;
#pragma unroll 4
    for (uint32_t b = q; b < nb; b += 4u) {
      const uint32_t c = code_hist[(size_t)b * 256 + d];
      all += c;
      before += b < blockIdx.x ? c : 0u;
    }
    part[0][q][d] = all;
    part[1][q][d] = before;
  }
#pragma unroll
  for (int k = 0; k < NW * 256 / kOrderNT; ++k) wcnt[0][t + (uint32_t)k * kOrderNT] = 0u;
  __syncthreads();
  if (t < 256) {
    uint32_t all = 0, before = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      all += part[0][q][t];
      before += part[1][q][t];
    }
    const uint32_t incl = wave_incl_scan(all);
    if (lane_id() == kWave - 1) red[w] = incl;
    base[t] = incl - all + before;
  }
  __syncthreads();
  if (t < 256)
    for (int k = 0; k < w; ++k) base[t] += red[k];
  const uint32_t tile = blockIdx.x * kOrderNT + t;
  const bool live = tile < sz.t_tot;
  const uint32_t code = live ? codes[tile] : 255u;
  const uint64_t eq = match_digit<8>(code, live);
  const uint32_t rank = (uint32_t)__popcll(eq & lanemask_lt());
  if (live && rank == 0) wcnt[w][code] = (uint32_t)__popcll(eq);
  __syncthreads();
  if (live) {
    uint32_t pos = base[code] + rank;
    for (int k = 0; k < w; ++k) pos += wcnt[k][code];
    ws.tile_order[pos] = tile;
  }
}

namespace {

// one workgroup scans up to one step of 16K words in about 4.5 us, two launches
// over many take 8 (64K words took it 20 us)
constexpr uint32_t kScanOneMax = 1u << 14;
constexpr uint32_t kScanFusedMax = 1024;    // chunks up to which each adds up the totals before it
constexpr uint32_t kRowWaveMax = 512;       // chunks up to which a wave scans a digit's row (two steps of 256)
constexpr uint32_t kOrderFusedMax = 512;    // blocks of tiles up to which the order takes one launch

// Exclusive scan of the first min(*count_dev, cap) words (cap if NULL) in
// place, part holding ceil(cap / 4096) words.
void scan_words(uint32_t *data, const uint32_t *count_dev, uint32_t cap, uint32_t *part, hipStream_t st) {
  if (cap == 0) return;
  if (cap <= kScanOneMax) {
    k_scan_one<<<1, 1024, 0, st>>>(data, count_dev, cap);
    return;
  }
  const uint32_t nb = cap / kScanChunk + (cap % kScanChunk != 0u);
  k_scan_reduce<<<nb, kScanNT, 0, st>>>(data, count_dev, cap, part);
  if (nb <= kScanFusedMax) {
    k_scan_down<true><<<nb, kScanNT, 0, st>>>(data, count_dev, cap, part);
    return;
  }
  k_scan_top<<<1, 1024, 0, st>>>(part, nb);
  k_scan_down<false><<<nb, kScanNT, 0, st>>>(data, count_dev, cap, part);
}

uint32_t chunks(uint32_t n, uint32_t chunk) { return std::max(1u, n / chunk + (n % chunk != 0u)); }

uint32_t rdx_chunk(uint32_t cap) { return (uint32_t)kRdxNT * (cap >= kRdxBig ? kRdxBigIPL : kRdxIPL); }

constexpr int kMaxBits = 11;  // widest digit

// Digit widths of a counting sort over `bits` key bits: one pass up to 11
// bits (2,040 tiles: 20 us, 32 in two), two 9- or 10-bit passes for 17 to 20
// rather than three, else 8-bit passes.  (Three passes of 10, 10 and 11 bits
// for the depths were no faster than four of 8: 99 against 93 us on 0.95M
// records, 746 against 700 on 12M; the wide scatters hold fewer waves.)
int sort_passes(int bits, int widths[4]) {
  if (bits > 8 && bits <= kMaxBits) {
    widths[0] = bits;
    return 1;
  }
  if (bits > 16 && bits <= 20) {
    widths[0] = widths[1] = (bits + 1) / 2;
    return 2;
  }
  const int passes = std::max(1, (bits + 7) / 8);
  for (int p = 0; p < passes; ++p) widths[p] = 8;
  return passes;
}

template <int IPL, int BITS>
void count_pass(const Ws &ws, uint32_t *hist, uint32_t nblk, const uint32_t *kin, const uint32_t *vin, uint32_t *kout,
                uint32_t *vout, const uint32_t *count_dev, uint32_t cap, int shift, uint32_t *aout, uint4 *rout,
                hipStream_t st) {
  const uint32_t pitch = (nblk + 3u) & ~3u;
  uint32_t *totals = ws.scan_part;
  k_digit_hist<IPL, BITS><<<nblk, kRdxNT, 0, st>>>(ws.scalars, kin, count_dev, cap, shift, pitch, hist);
  if (nblk > kRowWaveMax)
    k_digit_rows<true><<<1u << BITS, 256, 0, st>>>(ws.scalars, count_dev, cap, kRdxNT * IPL, pitch, hist, totals);
  else
    k_digit_rows<false><<<(1u << BITS) / 4, 256, 0, st>>>(ws.scalars, count_dev, cap, kRdxNT * IPL, pitch, hist,
                                                          totals);
  k_digit_scatter<IPL, BITS><<<nblk, kRdxNT, 0, st>>>(ws.scalars, kin, vin, kout, vout, count_dev, cap, shift, pitch,
                                                      hist, totals, ws.rec_rect, aout, rout);
}

// Stable sort of `cap` items, of which *count_dev (all if NULL) are live, by
// the low `bits` bits of their keys.  Input (k0, v0; v0 = NULL: values are
// the indices); pass p writes (kb, vb) for even p and (ka, va) for odd p,
// the last pass (out_k, out_v), one of the two, which must not be its own
// input.  (ka, va) may be the input itself.  With area_out the last pass also writes the
// tile-rectangle areas of the (record) values, and their tile records to
// rect_out, in sorted order.  hist: hist_words(cap, bits) words.
void counting_sort(const Ws &ws, uint32_t *hist, const uint32_t *count_dev, uint32_t cap, int bits, const uint32_t *k0,
                   const uint32_t *v0, uint32_t *ka, uint32_t *va, uint32_t *kb, uint32_t *vb, uint32_t *out_k,
                   uint32_t *out_v, uint32_t *area_out, uint4 *rect_out, hipStream_t st) {
  if (cap <= kMergeMax) {  // whole bytes of key bits: the keys hold none above `bits`
    const int digits = std::max(1, (bits + 7) / 8);
    const uint32_t runs = chunks(cap, kRunItems);
    if (runs == 1) {
      k_sort_runs<<<1, kRunNT, 0, st>>>(ws.scalars, k0, v0, out_k, out_v, count_dev, cap, digits, ws.rec_rect, area_out,
                                        rect_out);
      return;
    }
    // the runs go to whichever buffer is not the output
    uint32_t *rk = out_k == kb ? ka : kb, *rv = out_k == kb ? va : vb;
    k_sort_runs<<<runs, kRunNT, 0, st>>>(ws.scalars, k0, v0, rk, rv, count_dev, cap, digits, ws.rec_rect, nullptr,
                                         nullptr);
    k_merge_runs<<<chunks(cap, 256), 256, 0, st>>>(ws.scalars, rk, rv, out_k, out_v, count_dev, cap, ws.rec_rect,
                                                   area_out, rect_out);
    return;
  }
  const uint32_t chunk = rdx_chunk(cap);
  const uint32_t nblk = chunks(cap, chunk);
  int widths[4];
  const int passes = sort_passes(bits, widths);
  const uint32_t *kin = k0, *vin = v0;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const bool last = p == passes - 1;
    uint32_t *kout = last ? out_k : (p % 2 == 0 ? kb : ka);
    uint32_t *vout = last ? out_v : (p % 2 == 0 ? vb : va);
    uint32_t *aout = last ? area_out : nullptr;
    uint4 *rout = last ? rect_out : nullptr;
    const bool big = cap >= kRdxBig;
    switch (widths[p] * 2 + (big ? 1 : 0)) {
      case 16: count_pass<kRdxIPL, 8>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 17: count_pass<kRdxBigIPL, 8>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 18: count_pass<kRdxIPL, 9>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 19: count_pass<kRdxBigIPL, 9>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 20: count_pass<kRdxIPL, 10>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 21: count_pass<kRdxBigIPL, 10>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      case 22: count_pass<kRdxIPL, 11>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
      default: count_pass<kRdxBigIPL, 11>(ws, hist, nblk, kin, vin, kout, vout, count_dev, cap, shift, aout, rout, st); break;
    }
    shift += widths[p];
    kin = kout;
    vin = vout;
  }
}

int bit_width(uint32_t x) { return x == 0 ? 0 : 32 - __builtin_clz(x); }

// Digit histogram words of a counting sort of up to `cap` items by `bits`
// bits (none for the runs): at most cap + 4 * 2^11, as a pass of w bits has
// 2^w counts per chunk of at least 2048 items.
size_t hist_words(uint32_t cap, int bits) {
  if (cap <= kMergeMax) return 0;
  const size_t pitch = ((size_t)chunks(cap, rdx_chunk(cap)) + 3) & ~size_t(3);
  int widths[4];
  const int passes = sort_passes(bits, widths);
  size_t words = 0;
  for (int p = 0; p < passes; ++p) words = std::max(words, (size_t(1) << widths[p]) * pitch);
  return words;
}

int tile_bits(const Sizes &sz) { return std::max(1, bit_width(sz.t_tot - 1)); }

}  // namespace

// The histograms of the depth and tile sorts need no memory of their own:
// the depth sort's are in g2d, the tile sort's in the partials after the
// sort's own buffer, both written first by the backward.
BinningScratch binning_scratch(const Sizes &sz) {
  BinningScratch b;
  b.radix_hist = std::max(256 * (size_t)chunks(sz.t_tot, kOrderNT), hist_words(sz.t_tot, 8));
  const size_t scan = std::max<size_t>(sz.cap_rec, (size_t)sz.t_tot + 1);
  b.scan_part = (scan + kScanChunk - 1) / kScanChunk;
  if (std::max(std::max(sz.cap_rec, sz.cap_pairs), sz.t_tot) > kMergeMax)
    b.scan_part = std::max<size_t>(b.scan_part, size_t(1) << kMaxBits);  // a pass's digit totals
  return b;
}

// Records by depth bits (four passes, or runs in rec_tmp[2..3]): the last
// reads rec_tmp[2..3] and writes the order to rec_tmp[0..1] (record indices
// in rec_tmp[1]), the records' tile-rectangle areas to rec_tmp[4] and their
// tile records to the start of the backward's partials (free until the tile
// sort, at least 48 bytes per record), so that the emission reads them in
// order.
void launch_depth_sort(const Ws &ws, const Sizes &sz, hipStream_t st) {
  if (sz.cap_rec == 0) return;
  uint32_t *q[5];
  for (int k = 0; k < 5; ++k) q[k] = ws.rec_tmp + (size_t)k * sz.cap_rec;
  counting_sort(ws, reinterpret_cast<uint32_t *>(ws.g2d), ws.scalars + kNumRecords, sz.cap_rec, 32, ws.rec_zbits, nullptr, q[0], q[1], q[2], q[3], q[0],
                q[1], q[4], reinterpret_cast<uint4 *>(ws.partials), st);
}

void launch_binning(const ViewInfo *views, const Ws &ws, const Sizes &sz, hipStream_t st) {
  if (sz.t_tot == 0) return;
  const uint32_t *perm = ws.rec_tmp + sz.cap_rec;
  // areas -> pair offsets
  uint32_t *offs = ws.rec_tmp + 4 * (size_t)sz.cap_rec;
  scan_words(offs, ws.scalars + kNumRecords, sz.cap_rec, ws.scan_part, st);
  // (tile, record) ping-pong in pairs_tmp and in the backward's partials
  // (unused until the backward runs)
  uint32_t *ka = ws.pairs_tmp, *va = ka + sz.cap_pairs;
  uint32_t *kb = reinterpret_cast<uint32_t *>(ws.partials), *vb = kb + sz.cap_pairs;
  const uint32_t waves = sz.cap_rec / kWave + (sz.cap_rec % kWave != 0u);
  const uint32_t blocks = std::min<uint32_t>((waves + 3) / 4, 8192u);
  // the tile records in depth order, written by the depth sort's last pass
  const uint4 *srect = reinterpret_cast<const uint4 *>(ws.partials);
  k_emit<<<std::max(blocks, 1u), 256, 0, st>>>(ws, sz, perm, srect, offs, ka, va);
  const int bits = tile_bits(sz);
  int widths[4];
  const int passes = sort_passes(bits, widths);
  // the last pass reads (kb, vb) when the pass count is even, else (ka, va)
  uint32_t *sorted_tiles = (passes % 2 == 1 && sz.cap_pairs > kMergeMax) ? kb : ka;
  counting_sort(ws, vb + sz.cap_pairs + (sz.cap_pairs * 2u & 3u), ws.scalars + kNumPairs, sz.cap_pairs, bits, ka, va, ka, va, kb, vb, sorted_tiles, ws.tile_recs,
                nullptr, nullptr, st);
  // longest list first, by 8-bit length codes
  uint32_t *codes = ws.tile_tmp;
  const uint32_t tb = chunks(sz.t_tot, kOrderNT);
  if (sz.cap_pairs >= kRdxBig) {
    k_tile_ranges<true><<<tb, kOrderNT, 0, st>>>(ws, sz, sorted_tiles, codes, ws.radix_hist);
  } else {
    k_tile_bounds<<<chunks(sz.cap_pairs, 1024), 256, 0, st>>>(ws, sz, sorted_tiles);
    k_tile_ranges<false><<<tb, kOrderNT, 0, st>>>(ws, sz, sorted_tiles, codes, ws.radix_hist);
  }
  if (tb <= kOrderFusedMax) {
    k_tile_order<<<tb, kOrderNT, 0, st>>>(ws, sz, codes, ws.radix_hist);
  } else {  // the values are the tile ids
    uint32_t *unused = codes + sz.t_tot;
    counting_sort(ws, ws.radix_hist, nullptr, sz.t_tot, 8, codes, nullptr, codes, unused, codes, unused, unused, ws.tile_order, nullptr,
                  nullptr, st);
  }
}

// Exclusive scan of the list lengths: the CSR offsets of the tile lists
// (lists are contiguous in tile order), for the binning export.
__global__ void k_copy_counts(Ws ws, Sizes sz, uint32_t *__restrict__ csr) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < sz.t_tot) csr[t] = ws.tile_count[t];
  if (t == sz.t_tot) csr[t] = 0u;
}

void launch_tile_csr(const Ws &ws, const Sizes &sz, uint32_t *csr, hipStream_t st) {
  k_copy_counts<<<(sz.t_tot + 256) / 256, 256, 0, st>>>(ws, sz, csr);
  scan_words(csr, nullptr, sz.t_tot + 1, ws.scan_part, st);
}

}  // namespace gsr
