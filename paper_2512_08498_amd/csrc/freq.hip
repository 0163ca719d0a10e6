// Frequency-based scheduling (Sec. 3.3, "Frequency-based Scheduling",
// Eqs. 9-12): the frequency significance X(I) = sum over bins of the
// channel 2-norm of the unnormalised 2D DFT, for a batch of planar RGB images
// of arbitrary sizes; the n x n box downsampling of the LOD levels; and the
// per-frame ratios, level updates and ratio-weighted frame draws.
//
// X takes two passes over HBM.  Row pass: a workgroup packs two rows of a
// channel into one complex FFT (z = row i + i row i+1; the two are separated
// by the Hermitian symmetry of real inputs), three channels and one or more
// such pairs at once, and writes the half spectrum j = 0..W/2 of each channel
// transposed (column-major per channel, the pair's two values side by side),
// so the column pass reads contiguous columns.  Neighbouring pairs run on one
// XCD, so their transposed 16-byte writes meet in the same L2.  Column pass: a
// workgroup FFTs the three channels of one or more half-spectrum columns, adds
// |F|^2 over the channels per bin, and sums the square roots; columns
// 1..ceil(W/2)-1 count twice (their mirror W - j has the same magnitudes).  A
// last pass sums each image's columns in order.
//
// The FFT is Stockham's self-sorting mixed-radix form (radices 2, 3, 4, 5,
// 7 and the composites 6, 8, 9, 10, 12, 15, 16; see fft_plan), one stage per
// radix over all sequences of the workgroup at once, in one LDS buffer: the
// first stage's butterflies are loaded from global memory, and the column
// pass's last stage keeps its bins in registers.  The twiddles come from a
// table per list of radices computed in double precision at plan time, in
// the order in which the stages read them.
//
// What bounds the two passes is the LDS and the stages' latency, not HBM (the
// six 1600x900 views of a rig: 104 MB in, 104 MB out and in again).  They
// take 64 and 43 us there; with the blue row alone in its transform, a copy of
// the row and of the twiddles through LDS and the buffer behind generic
// pointers (flat instructions, 151 and 211 VGPRs) it was 115 and 119.
#include <cfloat>

#include "kernels.hpp"
#include "util.hpp"

namespace gsr {

namespace {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// multiply by -i
__device__ __forceinline__ float2 cmi(float2 a) { return make_float2(a.y, -a.x); }

// a / d for 0 <= a < 2^24, d >= 1, from a float reciprocal with one
// correction step each way (the float quotient is off by at most one).
__device__ __forceinline__ int fdiv(int a, int d, float inv) {
  int q = (int)((float)a * inv);
  q -= (q * d > a) ? 1 : 0;
  q += ((q + 1) * d <= a) ? 1 : 0;
  return q;
}

// exp(-2 pi i k / P) for k = 1 .. P - 1 (the forward sign).
template <int P>
struct Roots;
template <>
struct Roots<3> {
  static __device__ __forceinline__ float2 w(int k) {
    return k == 1 ? make_float2(-0.5f, -0.8660254037844386f) : make_float2(-0.5f, 0.8660254037844386f);
  }
};
template <>
struct Roots<5> {
  static __device__ __forceinline__ float2 w(int k) {
    switch (k) {
      case 1: return make_float2(0.30901699437494742f, -0.95105651629515357f);
      case 2: return make_float2(-0.80901699437494742f, -0.58778525229247313f);
      case 3: return make_float2(-0.80901699437494742f, 0.58778525229247313f);
      default: return make_float2(0.30901699437494742f, 0.95105651629515357f);
    }
  }
};
template <>
struct Roots<7> {
  static __device__ __forceinline__ float2 w(int k) {
    switch (k) {
      case 1: return make_float2(0.62348980185873353f, -0.78183148246802981f);
      case 2: return make_float2(-0.22252093395631440f, -0.97492791218182361f);
      case 3: return make_float2(-0.90096886790241913f, -0.43388373911755812f);
      case 4: return make_float2(-0.90096886790241913f, 0.43388373911755812f);
      case 5: return make_float2(-0.22252093395631440f, 0.97492791218182361f);
      default: return make_float2(0.62348980185873353f, 0.78183148246802981f);
    }
  }
};

// Composite radices P = A B, done in registers as B DFTs of size A, the
// twiddles exp(-2 pi i a b / P), then A DFTs of size B (Cooley-Tukey with
// n = B n1 + n2, k = k1 + A k2), so one Stockham stage covers two factors.
template <int P>
struct Split {
  static constexpr int A = 1, B = P;
};
template <> struct Split<6> { static constexpr int A = 2, B = 3; };
template <> struct Split<8> { static constexpr int A = 4, B = 2; };
template <> struct Split<9> { static constexpr int A = 3, B = 3; };
template <> struct Split<10> { static constexpr int A = 2, B = 5; };
template <> struct Split<12> { static constexpr int A = 4, B = 3; };
template <> struct Split<15> { static constexpr int A = 3, B = 5; };
template <> struct Split<16> { static constexpr int A = 4, B = 4; };

// cos and sin at compile time: Taylor series in double on |x| <= pi (30
// terms, far below float resolution).
constexpr double ct_sin(double x) {
  double t = x, s = x;
  for (int k = 1; k < 30; ++k) {
    t *= -x * x / (double)((2 * k) * (2 * k + 1));
    s += t;
  }
  return s;
}
constexpr double ct_cos(double x) {
  double t = 1.0, s = 1.0;
  for (int k = 1; k < 30; ++k) {
    t *= -x * x / (double)((2 * k - 1) * (2 * k));
    s += t;
  }
  return s;
}

// cos and sin of 2 pi m / P, m = 0 .. P - 1.
template <int P>
struct TwiddleTable {
  float c[P], s[P];
  constexpr TwiddleTable() : c(), s() {
    constexpr double kPi = 3.14159265358979323846;
    for (int m = 0; m < P; ++m) {
      double x = 2.0 * kPi * m / P;
      if (x > kPi) x -= 2.0 * kPi;
      c[m] = (float)ct_cos(x);
      s[m] = (float)ct_sin(x);
    }
  }
};

template <int P>
__device__ __forceinline__ void dft(float2 *v);

template <int P>
__device__ __forceinline__ void dft_composite(float2 *v) {
  constexpr int A = Split<P>::A, B = Split<P>::B;
  constexpr TwiddleTable<P> tw{};
  float2 t[P];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    float2 u[A];
#pragma unroll
    for (int a = 0; a < A; ++a) u[a] = v[b + B * a];
    dft<A>(u);
#pragma unroll
    for (int a = 0; a < A; ++a) {
      const int m = (a * b) % P;  // u exp(-2 pi i m / P) = u (c - i s)
      t[a * B + b] = m == 0 ? u[a]
                            : make_float2(u[a].x * tw.c[m] + u[a].y * tw.s[m], u[a].y * tw.c[m] - u[a].x * tw.s[m]);
    }
  }
#pragma unroll
  for (int a = 0; a < A; ++a) dft<B>(t + a * B);
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) v[a + A * b] = t[a * B + b];
}

// In-register radix-P DFT with the forward sign (P = 1: nothing).  Radices 3
// and 5 use the symmetric forms: with s_k = x_k + x_{P-k} and d_k = x_k - x_{P-k},
// X_q = x_0 + sum_k cos(2 pi k q / P) s_k - i sum_k sin(2 pi k q / P) d_k.
template <int P>
__device__ __forceinline__ void dft(float2 *v) {
  if constexpr (P == 1) {
  } else if constexpr (Split<P>::A > 1) {
    dft_composite<P>(v);
  } else if constexpr (P == 3) {
    constexpr float s1 = 0.86602540378443865f;  // sin(2 pi / 3)
    const float2 s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const float2 a = make_float2(v[0].x - 0.5f * s.x, v[0].y - 0.5f * s.y);
    const float2 b = make_float2(s1 * d.y, -s1 * d.x);  // -i sin(2 pi / 3) d
    v[0] = cadd(v[0], s);
    v[1] = cadd(a, b);
    v[2] = csub(a, b);
  } else if constexpr (P == 5) {
    constexpr float c1 = 0.30901699437494742f, c2 = -0.80901699437494742f;  // cos(2 pi / 5), cos(4 pi / 5)
    constexpr float s1 = 0.95105651629515357f, s2 = 0.58778525229247313f;   // sin(2 pi / 5), sin(4 pi / 5)
    const float2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]);
    const float2 t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
    const float2 a1 = make_float2(v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y);
    const float2 a2 = make_float2(v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y);
    const float2 b1 = make_float2(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y);
    const float2 b2 = make_float2(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y);
    v[0] = cadd(v[0], cadd(t1, t2));
    v[1] = cadd(a1, cmi(b1));
    v[4] = csub(a1, cmi(b1));
    v[2] = cadd(a2, cmi(b2));
    v[3] = csub(a2, cmi(b2));
  } else if constexpr (P == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (P == 4) {
    const float2 a = v[0], b = v[1], c = v[2], d = v[3];
    const float2 s0 = cadd(a, c), s1 = csub(a, c), s2 = cadd(b, d), s3 = cmi(csub(b, d));
    v[0] = cadd(s0, s2);
    v[1] = cadd(s1, s3);
    v[2] = csub(s0, s2);
    v[3] = csub(s1, s3);
  } else {
    float2 o[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      float2 acc = v[0];
#pragma unroll
      for (int r = 1; r < P; ++r) {
        const int e = (q * r) % P;
        acc = cadd(acc, e == 0 ? v[r] : cmul(v[r], Roots<P>::w(e)));
      }
      o[q] = acc;
    }
#pragma unroll
    for (int q = 0; q < P; ++q) v[q] = o[q];
  }
}


// The workgroup's buffer: an LDS pointer of its own kind, so that the stages
// take ds_ instructions.
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2f Lds2;

__device__ __forceinline__ float2 get(const Lds2 *p) {
  const v2f t = *p;
  return make_float2(t.x, t.y);
}
__device__ __forceinline__ void put(Lds2 *p, float2 x) {
  v2f t;
  t.x = x.x;
  t.y = x.y;
  *p = t;
}

// A radix-P Stockham stage over `cnt` sequences of length N stored one after
// the other.  Butterfly b (sequence b / m, index j = b mod m, m = N / P)
// reads elements j + r m, multiplies by the twiddles exp(-2 pi i k r / (Ns P))
// (k = j mod Ns; table entry (r - 1) Ns + k of the stage), transforms, and
// writes (j / Ns) Ns P + k + q Ns.  The stages are inlined: as calls they saved
// registers to scratch.

// First stage (Ns = 1, no twiddles) of the row pass: sequence 3 p + c packs
// rows row0 + 2 p and the next of channel c (zeros past the last row).
template <int P, int T>
__device__ __forceinline__ void rows_in(Lds2 *buf, const float *img, int W, int H, int row0, int cnt) {
  const int m = W / P, total = cnt * m;
  const float inv_m = 1.0f / (float)m;
  for (int b = threadIdx.x; b < total; b += T) {
    const int seq = fdiv(b, m, inv_m), j = b - seq * m, pair = seq / 3, c = seq - 3 * pair;
    const int row = row0 + 2 * pair;
    const float *src = img + ((int64_t)c * H + row) * W + j;
    const bool two = row + 1 < H;
    float2 v[P];
#pragma unroll
    for (int r = 0; r < P; ++r) v[r] = make_float2(src[r * m], two ? src[W + r * m] : 0.0f);
    dft<P>(v);
#pragma unroll
    for (int q = 0; q < P; ++q) put(buf + seq * W + j * P + q, v[q]);
  }
}

// First stage of the column pass: sequence 3 k + c is column col0 + k of
// channel c.
template <int P, int T>
__device__ __forceinline__ void cols_in(Lds2 *buf, const float2 *inter, int H, int pitch, int half, int col0,
                                                  int cnt) {
  const int m = H / P, total = cnt * m;
  const float inv_m = 1.0f / (float)m;
  for (int b = threadIdx.x; b < total; b += T) {
    const int seq = fdiv(b, m, inv_m), j = b - seq * m, k = seq / 3, c = seq - 3 * k;
    const float2 *src = inter + ((int64_t)c * half + col0 + k) * pitch + j;
    float2 v[P];
#pragma unroll
    for (int r = 0; r < P; ++r) v[r] = src[r * m];
    dft<P>(v);
#pragma unroll
    for (int q = 0; q < P; ++q) put(buf + seq * H + j * P + q, v[q]);
  }
}

// A later stage in LDS.  All butterflies of the thread are loaded and
// transformed before the barrier, then stored, so one buffer suffices.
template <int P, int T, int MAXE>
__device__ __forceinline__ void stage(Lds2 *buf, int N, int cnt, int Ns, const float2 *tw) {
  int t0 = threadIdx.x;
  asm volatile("" : "+v"(t0));  // keeps every radix's indices from being computed ahead of the loop over the stages
  constexpr int kMaxB = (MAXE / P + T - 1) / T;
  const int m = N / P, total = cnt * m;
  const float inv_m = 1.0f / (float)m, inv_ns = 1.0f / (float)Ns;
  float2 v[kMaxB][P];
  int dst[kMaxB];
#pragma unroll
  for (int i = 0; i < kMaxB; ++i) {
    const int b = t0 + i * T;
    if (b < total) {
      const int seq = fdiv(b, m, inv_m), j = b - seq * m;
      const int jq = fdiv(j, Ns, inv_ns), k = j - jq * Ns;
      const Lds2 *src = buf + seq * N + j;
      v[i][0] = get(src);
#pragma unroll
      for (int r = 1; r < P; ++r) v[i][r] = cmul(get(src + r * m), tw[(r - 1) * Ns + k]);
      dft<P>(v[i]);
      dst[i] = seq * N + jq * Ns * P + k;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kMaxB; ++i) {
    const int b = t0 + i * T;
    if (b < total) {
#pragma unroll
      for (int q = 0; q < P; ++q) put(buf + dst[i] + q * Ns, v[i][q]);
    }
  }
}

// Last stage (Ns = m) of the column pass: butterfly b of `cols` columns takes
// the three channels in turn and leaves the sum of its bins' norms in part[b].
template <int P, int T>
__device__ __forceinline__ void cols_out(const Lds2 *buf, int H, int cols, const float2 *tw,
                                                   __attribute__((address_space(3))) float *part) {
  const int m = H / P, total = cols * m;
  const float inv_m = 1.0f / (float)m;
  for (int b = threadIdx.x; b < total; b += T) {
    const int k = fdiv(b, m, inv_m), j = b - k * m;
    const Lds2 *src = buf + 3 * k * H + j;
    float2 w[P];
#pragma unroll
    for (int r = 1; r < P; ++r) w[r] = tw[(r - 1) * m + j];
    float acc[P];
#pragma unroll
    for (int q = 0; q < P; ++q) acc[q] = 0.0f;
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
      float2 v[P];
      v[0] = get(src + c * H);
#pragma unroll
      for (int r = 1; r < P; ++r) v[r] = cmul(get(src + c * H + r * m), w[r]);
      dft<P>(v);
#pragma unroll
      for (int q = 0; q < P; ++q) acc[q] += v[q].x * v[q].x + v[q].y * v[q].y;
    }
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < P; ++q) s += sqrtf(acc[q]);
    part[b] = s;
  }
}

template <int P>
struct Radix {
  static constexpr int value = P;
};

// Calls f with the radix as a compile-time constant.
template <bool SMALL, class F>
__device__ __forceinline__ void with_radix(int p, const F &f) {
  switch (p) {
    case 16: f(Radix<16>()); break;
    case 15: f(Radix<15>()); break;
    case 12: f(Radix<12>()); break;
    case 10: f(Radix<10>()); break;
    case 9: f(Radix<9>()); break;
    case 8: f(Radix<8>()); break;
    case 7: f(Radix<7>()); break;
    case 6: f(Radix<6>()); break;
    case 5: f(Radix<5>()); break;
    default:
      if constexpr (SMALL) {
        if (p == 4) f(Radix<4>());
        else if (p == 3) f(Radix<3>());
        else if (p == 2) f(Radix<2>());
        else f(Radix<1>());
      }
  }
}

// The stages fac[1 .. last) between a first one and, for the column pass, a
// last one.  Returns Ns behind them.  A stage's table follows those of the
// stages before, whose sizes add up to Ns - fac[0].
template <int T, int MAXE>
__device__ __forceinline__ int middle_stages(Lds2 *buf, int N, int cnt, const uint8_t *__restrict__ fac, int last,
                                             const float2 *__restrict__ tw) {
  int Ns = fac[0];
  __syncthreads();
  for (int s = 1; s < last; ++s) {
    const float2 *t = tw + (Ns - fac[0]);
    with_radix<false>(fac[s], [&](auto p) { stage<decltype(p)::value, T, MAXE>(buf, N, cnt, Ns, t); });
    __syncthreads();
    Ns *= fac[s];
  }
  return Ns;
}

__device__ __forceinline__ int find_image(const FreqImg *imgs, int n, int64_t idx, bool rows) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((rows ? imgs[mid].row_group : imgs[mid].col_group) <= idx) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Deterministic sum over a workgroup of NW waves: butterfly per wave, then
// the waves in order; the result is valid in every thread.
template <int NW>
__device__ __forceinline__ double block_sum(double x, double *red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double t = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t += red[w];
  return t;
}

__global__ __launch_bounds__(kFreqRowThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_fft_rows(
    const float *__restrict__ images, const FreqImg *__restrict__ imgs, int n_imgs, int64_t n_groups,
    const float2 *__restrict__ tw_all, float2 *__restrict__ inter) {
  constexpr int T = kFreqRowThreads;
  extern __shared__ float2 lds[];
  Lds2 *buf = (Lds2 *)lds;
  const int64_t group = xcd_tile(blockIdx.x, gridDim.x);
  if (group >= n_groups) return;
  const FreqImg *ip = imgs + find_image(imgs, n_imgs, group, true);
  const FreqImg im = *ip;
  const int W = im.w, H = im.h, half = W / 2 + 1, pitch = freq_pitch(H);
  const int row0 = (int)(group - im.row_group) * 2 * im.pairs;
  const int pairs = min(im.pairs, (H - row0 + 1) / 2), cnt = 3 * pairs;
  with_radix<true>(ip->fac_w[0], [&](auto p) { rows_in<decltype(p)::value, T>(buf, images + im.pix_off, W, H, row0, cnt); });
  middle_stages<T, kFreqRowElems>(buf, W, cnt, ip->fac_w, im.nfac_w, tw_all + im.tw_w);
  float2 *out = inter + im.inter_off;
  const int total = half * pairs;
  const float inv_p = 1.0f / (float)pairs;
  for (int c = 0; c < 3; ++c)
    for (int b = threadIdx.x; b < total; b += T) {
      const int j = pairs == 1 ? b : fdiv(b, pairs, inv_p), pair = b - j * pairs;
      const Lds2 *z = buf + (3 * pair + c) * W;
      const float2 p = get(z + j), q = get(z + (j == 0 ? 0 : W - j));
      // F_i = (Z(j) + conj Z(-j)) / 2,  F_i+1 = (Z(j) - conj Z(-j)) / 2i
      *reinterpret_cast<float4 *>(out + ((int64_t)c * half + j) * pitch + row0 + 2 * pair) =
          make_float4(0.5f * (p.x + q.x), 0.5f * (p.y - q.y), 0.5f * (p.y + q.y), -0.5f * (p.x - q.x));
    }
}

__global__ __launch_bounds__(kFreqColThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_fft_cols(
    const FreqImg *__restrict__ imgs, int n_imgs, int64_t n_groups, const float2 *__restrict__ tw_all,
    const float2 *__restrict__ inter, float *__restrict__ col_sum) {
  constexpr int T = kFreqColThreads;
  extern __shared__ float2 lds[];
  Lds2 *buf = (Lds2 *)lds;
  const int64_t group = blockIdx.x;
  if (group >= n_groups) return;
  const FreqImg *ip = imgs + find_image(imgs, n_imgs, group, false);
  const FreqImg im = *ip;
  const int W = im.w, H = im.h, half = W / 2 + 1;
  const int col0 = (int)(group - im.col_group) * im.cols, cols = min(im.cols, half - col0), cnt = 3 * cols;
  with_radix<true>(ip->fac_h[0], [&](auto p) {
    cols_in<decltype(p)::value, T>(buf, inter + im.inter_off, H, freq_pitch(H), half, col0, cnt);
  });
  const float2 *tw = tw_all + im.tw_h;
  const int Ns = middle_stages<T, 3 * kFreqMaxN>(buf, H, cnt, ip->fac_h, im.nfac_h - 1, tw);
  auto *part = (__attribute__((address_space(3))) float *)(buf + cnt * H);
  with_radix<true>(ip->fac_h[im.nfac_h - 1],
             [&](auto p) { cols_out<decltype(p)::value, T>(buf, H, cols, tw + (Ns - ip->fac_h[0]), part); });
  __syncthreads();
  // a wave per column: lane l adds values l, l + 64, ..., then the lanes
  const int lane = threadIdx.x & 63;
  for (int k = threadIdx.x >> 6; k < cols; k += T / 64) {
    float s = 0.0f;
    for (int i = lane; i < Ns; i += 64) s += part[k * Ns + i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    const int j = col0 + k;
    const bool single = j == 0 || (W % 2 == 0 && j == W / 2);
    if (lane == 0) col_sum[im.col_base + j] = single ? s : 2.0f * s;
  }
}

// X of each image: its columns' sums in column order (thread t takes the
// columns t mod 256 in order, then the fixed block sum), in double precision:
// the sum's own rounding had been most of X's error.
__global__ __launch_bounds__(256) void k_freq_final(const FreqImg *__restrict__ imgs,
                                                    const float *__restrict__ col_sum, float *__restrict__ X) {
  __shared__ double red[4];
  const FreqImg im = imgs[blockIdx.x];
  const int half = im.w / 2 + 1;
  double s = 0.0;
  for (int j = threadIdx.x; j < half; j += blockDim.x) s += col_sum[im.col_base + j];
  const double total = block_sum<4>(s, red);
  if (threadIdx.x == 0) X[blockIdx.x] = (float)total;
}

// Box average over n x n blocks; one thread per output value, the block's
// values added row by row.  I: 32-bit indices where they suffice (64-bit
// divisions cost more than the reads).  N: n where it is known, so that its
// reads are issued together.
template <typename I, int N>
__global__ __launch_bounds__(256) void k_downsample(const float *__restrict__ src, int W, int H, int n_,
                                                    float *__restrict__ dst) {
  const int n = N ? N : n_;
  const I w = (I)(W / n), h = (I)(H / n);
  const I total = 3 * w * h;
  const I idx = (I)blockIdx.x * (I)blockDim.x + (I)threadIdx.x;
  if (idx >= total) return;
  const I row = idx / w, x = idx - row * w;
  const I c = row / h, y = row - c * h;
  const float *p = src + ((int64_t)c * H + (int64_t)y * n) * W + (int64_t)x * n;
  float s = 0.0f;
#pragma unroll
  for (int dy = 0; dy < n; ++dy)
#pragma unroll
    for (int dx = 0; dx < n; ++dx) s += p[(int64_t)dy * W + dx];
  dst[idx] = s / (float)(n * n);
}

// Ratios, level updates and frame draws of one scheduling step (single
// workgroup; the prefix sums of the weights are taken by one thread in frame
// order, in float32, so the draws are reproducible bit for bit).
__global__ __launch_bounds__(256) void k_freq_schedule(const float *__restrict__ x_gt,
                                                       const float *__restrict__ x_gt_level,
                                                       const float *__restrict__ x_render, int F, float tau_f,
                                                       int32_t *__restrict__ levels, const float *__restrict__ u,
                                                       int n_picks, float *__restrict__ r_out,
                                                       float *__restrict__ rp_out, int32_t *__restrict__ picks) {
  extern __shared__ float cdf[];
  const float cap = FLT_MAX / (float)(2 * F);  // F capped weights cannot overflow
  for (int f = threadIdx.x; f < F; f += blockDim.x) {
    const float r = x_gt[f] / x_render[f];
    const float rp = x_gt_level ? x_gt_level[f] / x_render[f] : __builtin_nanf("");
    if (r_out) r_out[f] = r;
    if (rp_out) rp_out[f] = rp;
    if (levels && rp < tau_f && levels[f] > 0) levels[f] -= 1;
    cdf[f] = isnan(r) ? 0.0f : fmaxf(fminf(r, cap), 0.0f);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float acc = 0.0f;
    for (int f = 0; f < F; ++f) {
      acc = acc + cdf[f];
      cdf[f] = acc;
    }
  }
  __syncthreads();
  if (!picks) return;
  const float total = cdf[F - 1];
  for (int b = threadIdx.x; b < n_picks; b += blockDim.x) {
    const float ub = u[b];
    int f;
    if (!(total > 0.0f)) {
      f = (int)(ub * (float)F);
      f = f < F - 1 ? f : F - 1;
      f = f > 0 ? f : 0;
    } else {
      const float target = ub * total;
      int lo = 0, hi = F - 1;  // first f with cdf[f] > target, else F - 1
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cdf[mid] > target) hi = mid;
        else lo = mid + 1;
      }
      f = lo;
    }
    picks[b] = f;
  }
}

}  // namespace

void launch_freq_significance(const float *images, const FreqImg *imgs, int n_imgs, int64_t row_groups,
                              int64_t col_groups, uint32_t lds_rows, uint32_t lds_cols, const float2 *tw, float2 *inter,
                              float *col_sum, float *X, hipStream_t st) {
  if (n_imgs == 0) return;
  const uint32_t grid = tile_grid((uint32_t)row_groups);
  k_fft_rows<<<grid, kFreqRowThreads, lds_rows, st>>>(images, imgs, n_imgs, row_groups, tw, inter);
  k_fft_cols<<<(unsigned)col_groups, kFreqColThreads, lds_cols, st>>>(imgs, n_imgs, col_groups, tw, inter, col_sum);
  k_freq_final<<<(unsigned)n_imgs, 256, 0, st>>>(imgs, col_sum, X);
}

void launch_downsample(const float *src, int W, int H, int n, float *dst, hipStream_t st) {
  const int64_t total = 3ll * (W / n) * (H / n);
  if (total == 0) return;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  if (total >= (int64_t(1) << 31))
    k_downsample<int64_t, 0><<<blocks, 256, 0, st>>>(src, W, H, n, dst);
  else if (n == 2)
    k_downsample<uint32_t, 2><<<blocks, 256, 0, st>>>(src, W, H, n, dst);
  else
    k_downsample<uint32_t, 0><<<blocks, 256, 0, st>>>(src, W, H, n, dst);
}

void launch_freq_schedule(const float *x_gt, const float *x_gt_level, const float *x_render, int F, float tau_f,
                          int32_t *levels, const float *u, int n_picks, float *r, float *rp, int32_t *picks,
                          hipStream_t st) {
  if (F == 0) return;
  k_freq_schedule<<<1, 256, (size_t)F * sizeof(float), st>>>(x_gt, x_gt_level, x_render, F, tau_f, levels, u,
                                                             n_picks, r, rp, picks);
}

}  // namespace gsr
