// Frequency-band decomposition of the calibration disagreement: the guided
// difference d = p_S - p_L (Eqs. 1, 4) on the C x F x H x W latent, read
// straight from the two models' patch-token velocities, is transformed with
// orthonormal DFTs (spatially over (H, W) per (c, f) slice, temporally over F
// per (c, h, w) series) and its energy split into low / mid / high bands of
// the normalised frequency nu = 2|k'|/n (k' the signed frequency index):
// low nu < 1/3, mid nu < 2/3, high otherwise, the spatial nu being the radius
// over (H, W).  Band membership is decided in integer arithmetic.
//
// Passes (all on the caller's stream):
//   band_temporal the F-point DFTs of 256 (c, h, w) series a block; the common
//                 layout also leaves d itself, one 2 x 2 patch of a channel per 16
//                 bytes in (frame, channel, token) order
//   band_spatial  64 columns k_w of one (c, f) slice's 2D DFT a block, from that (the
//                 velocities interleave a token's channels: each slice read straight
//                 from them takes 16 of every 256 bytes)
//   each leaves a block's three band energies (fp64) as a partial
//   band_finish   partials summed in a fixed order -> 6 energies (and scores)
// The DFTs are products with the axis' cosine and sine matrices on
// v_mfma_f32_16x16x4_f32 (float32 products and sums), whose entries are looked up
// in LDS tables exp(-2 pi i m / n) (fp64 -> fp32) at (k x) mod n; each frequency's
// energy is freed of its entries' rounding (freq_sums).  The input is real, so k_w
// (temporal: k_f) runs to n / 2 only, the rest being the conjugates at -k, and row
// k_h and row H - k_h come from the same four products.
#include <math.h>

#include "common.h"
#include "kernels.h"

namespace track {

namespace {

constexpr int BAND_THREADS = 256;
constexpr int BAND_COLS = 64;     // columns k_w per spatial block, 16 a wave
constexpr int BAND_XCH = 128;     // latent columns staged at a time
constexpr int BAND_XLD = BAND_XCH + 4;  // LDS row stride: 4 mod 8 floats, so 16 rows' 16-byte reads hit all banks
constexpr int BAND_MAX_W = 1024;  // twiddle table bound
constexpr int BAND_MAX_H = 256;   // LDS bound of a staged chunk, and the accumulators of 16 row blocks
constexpr int BAND_MAX_F = 64;    // temporal kernel LDS bound
constexpr int BAND_MAX_DIVS = 32;  // divisors of a length up to 1024 (840 has 32, itself among them)
constexpr int BAND_EXTRA = 2;      // first blocks of the temporal pass, which do the spatial axes' sums

inline unsigned blocks_for(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }
inline size_t align_256(size_t v) { return (v + 255) & ~(size_t)255; }

struct BandShape {
  int C, F, H, W, pt, ph, pw;
  int Hp, Wp, P;
};

// Offset of latent element (c, f, h, w) in the patch-token layout [L][P].
__device__ __forceinline__ int64_t tok_offset(const BandShape& s, int c, int f, int h, int w) {
  const int64_t l = ((int64_t)(f / s.pt) * s.Hp + h / s.ph) * s.Wp + w / s.pw;
  const int e = ((c * s.pt + f % s.pt) * s.ph + h % s.ph) * s.pw + w % s.pw;
  return l * s.P + e;
}

// Guided difference p_S - p_L at token-layout offset o (Eq. 1 per model).
__device__ __forceinline__ float guided_diff(const float* __restrict__ vL, const float* __restrict__ vS, int64_t n,
                                             int B, float w, int64_t o) {
  const float cL = vL[o], cS = vS[o];
  if (B == 2) {
    const float pL = fmaf(w, cL - vL[n + o], vL[n + o]);
    const float pS = fmaf(w, cS - vS[n + o], vS[n + o]);
    return pS - pL;
  }
  return cS - cL;
}

// |k'| of frequency index k on an axis of length n.
__device__ __forceinline__ int64_t fold(int k, int n) { return k <= n / 2 ? k : n - k; }

__device__ __forceinline__ int axis_band(int k, int n) {
  const int64_t a = fold(k, n);
  return 6 * a < n ? 0 : (3 * a < n ? 1 : 2);
}

// nu^2 / 4 * H^2 W^2 = a_h^2 W^2 + a_w^2 H^2 against (1/3)^2 and (2/3)^2.
__device__ __forceinline__ int spatial_band(int kh, int kw, int H, int W) {
  const int64_t ah = fold(kh, H), aw = fold(kw, W);
  const int64_t s = ah * ah * W * W + aw * aw * H * H;
  const int64_t hw2 = (int64_t)H * H * W * W;
  return 36 * s < hw2 ? 0 : (9 * s < hw2 ? 1 : 2);
}

// Block-wide sum of three doubles per thread; thread 0 writes them to out[0..2].
__device__ __forceinline__ void block_sum3(double a0, double a1, double a2, double* __restrict__ out) {
  __shared__ double red[3][BAND_THREADS / 64];
  a0 = wave_sum_d(a0);
  a1 = wave_sum_d(a1);
  a2 = wave_sum_d(a2);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wv] = a0;
    red[1][wv] = a1;
    red[2][wv] = a2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int b = 0; b < 3; ++b) {
      double acc = 0.0;
      for (int i = 0; i < BAND_THREADS / 64; ++i) acc += red[b][i];
      out[b] = acc;
    }
  }
}

// (a + b) mod n for a, b < n
__device__ __forceinline__ uint32_t add_mod(uint32_t a, uint32_t b, uint32_t n) { return min(a + b, a + b - n); }

__device__ __forceinline__ float2 twiddle(int m, int n) {
  double sn, cs;
  sincospi(2.0 * m / n, &sn, &cs);
  return make_float2((float)cs, (float)-sn);
}

__device__ __forceinline__ void fill_twiddles(float2* __restrict__ tw, int n) {
  for (int m = threadIdx.x; m < n; m += BAND_THREADS) tw[m] = twiddle(m, n);
}

// |t|^2 - 1
__device__ __forceinline__ float deviation(float2 t) {
  return (float)fma((double)t.x, (double)t.x, fma((double)t.y, (double)t.y, -1.0));
}

// A frequency's energy is divided by the sum of |t|^2 over the n table entries t that its
// transform took, n + dsum, in place of n: the entries' float32 rounding scales the energy
// by their mean |t|^2, which would be the largest error of the transforms (8e-9 to 3e-8 of
// the energies over latents of 16 - 90 rows, 4e-10 to 8e-9 with it taken out, for 1 of the
// pass' 52 us on the video latent).  One factor for a whole axis would do as well on
// average, but puts 1e-8 on the mean, whose entries are exact.  Frequency k takes the
// multiples of g = gcd(k, n), each g times, so one sum per divisor of n serves all.
__device__ __forceinline__ void freq_sums(float* __restrict__ dsum, int n) {
  __shared__ float dev[BAND_MAX_W];
  __shared__ int divs[BAND_MAX_DIVS], ndivs;
  if (threadIdx.x == 0) ndivs = 0;
  __syncthreads();
  for (int m = threadIdx.x; m < n; m += BAND_THREADS) dev[m] = deviation(twiddle(m, n));
  for (int d = 1 + threadIdx.x; d <= n / 2; d += BAND_THREADS)
    if (n % d == 0) divs[atomicAdd(&ndivs, 1)] = d;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x >> 6; i < ndivs; i += BAND_THREADS / 64) {
    const int d = divs[i];
    float e = 0.0f;
    for (int m = lane * d; m < n; m += 64 * d) e += dev[m];
    e = (float)d * wave_sum(e);
    if (lane == 0) dsum[d] = e;
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= n / 2; k += BAND_THREADS) {
    int g = n, r = k;
    while (r) {
      const int t = g % r;
      g = r;
      r = t;
    }
    if (g != k) dsum[k] = g == n ? 0.0f : dsum[g];
  }
}

// The table of the F axis (F <= 64 entries) and the sums of its frequencies: every lane of
// a 16-lane group takes one frequency and a quarter of its entries.
__device__ __forceinline__ void fill_temporal(float2* __restrict__ tw, float* __restrict__ dev, float* __restrict__ dsum,
                                              uint32_t n) {
  if (threadIdx.x < n) {
    const float2 t = twiddle(threadIdx.x, n);
    tw[threadIdx.x] = t;
    dev[threadIdx.x] = deviation(t);
  }
  __syncthreads();
  const uint32_t k = threadIdx.x >> 6 << 4 | (threadIdx.x & 15), g = (threadIdx.x >> 4) & 3;
  const uint32_t k1 = min(k, n - 1), k2 = add_mod(k1, k1, n), step = add_mod(k2, k2, n);
  uint32_t m = (g & 2) ? k2 : 0;
  if (g & 1) m = add_mod(m, k1, n);
  float e = 0.0f;
#pragma unroll 8
  for (uint32_t x = g; x < n; x += 4) {
    e += dev[m];
    m = add_mod(m, step, n);
  }
  e += __shfl_xor(e, 16);
  e += __shfl_xor(e, 32);
  dsum[k] = e;  // (the same from all four groups)
  __syncthreads();
}

// 1 / (n + dsum) for rn = 1 / n; dsum is some 1e-8 of n, so its square is out of reach.
__device__ __forceinline__ double inv_sum(double rn, float dsum) { return fma(-(double)dsum * rn, rn, rn); }

__device__ __forceinline__ f32x4 guided_diff4(const float* __restrict__ vL, const float* __restrict__ vS, int64_t n,
                                              int B, float w, int64_t o) {
  const f32x4 cL = *(const f32x4*)(vL + o), cS = *(const f32x4*)(vS + o);
  f32x4 d;
  if (B == 2) {
    const f32x4 uL = *(const f32x4*)(vL + n + o), uS = *(const f32x4*)(vS + n + o);
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = fmaf(w, cS[j] - uS[j], uS[j]) - fmaf(w, cL[j] - uL[j], uL[j]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = cS[j] - cL[j];
  }
  return d;
}

__device__ __forceinline__ void add_band(double (&acc)[3], int b, double e) {
  acc[0] += b == 0 ? e : 0.0;
  acc[1] += b == 1 ? e : 0.0;
  acc[2] += b == 2 ? e : 0.0;
}

// Spatial block: slice (c, f), columns k_w = 64 kg .. + 63, 16 a wave.  The slice
// (up to BAND_XCH columns at a time, rows and columns padded with zeros) is staged
// in LDS as the MFMA "A" operand; a wave's row DFTs for all rows stay in its
// accumulators (lane: column k_w, rows 16 b + 4 g + r), which are the "B" operand of
// the column DFT as they are.  Slices are numbered frame by frame over the XCDs, so
// that those of one frame are read through one L2.
template <int HB>
__global__ __launch_bounds__(BAND_THREADS) void band_spatial_kernel(BandShape s, int B, float w,
                                                                    const float* __restrict__ vL,
                                                                    const float* __restrict__ vS, int64_t n,
                                                                    const f32x4* __restrict__ diff,
                                                                    const float* __restrict__ dsum, int kwg,
                                                                    double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float sd[16 * HB][BAND_XLD];
  __shared__ float2 twW[BAND_MAX_W], twH[BAND_MAX_H];
  __shared__ float sumH[BAND_MAX_H / 2 + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int jq = lane & 15, g = lane >> 4;
  const int id = xcd_remap(blockIdx.x, gridDim.x);
  const int f = id / (s.C * kwg), c = id / kwg % s.C, kg = id % kwg;
  // (the W / 2 + 1 sums of the rows' frequencies, then the H / 2 + 1 of the columns')
  for (int k = threadIdx.x; k <= s.H / 2; k += BAND_THREADS) sumH[k] = dsum[s.W / 2 + 1 + k];
  fill_twiddles(twW, s.W);
  fill_twiddles(twH, s.H);
  const uint32_t W = s.W, H = s.H;
  const int kw0 = (kg * 4 + wave) * 16, kw = kw0 + jq;
  const bool live = kw0 <= s.W / 2;  // wave-uniform
  const float sumW = dsum[min(kw, s.W / 2)];
  f32x4 yr[HB], yi[HB];
#pragma unroll
  for (int b = 0; b < HB; ++b) yr[b] = yi[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t step16 = (16u * kw) % W;
  for (int x0 = 0; x0 < s.W; x0 += BAND_XCH) {
    const int xc = min(BAND_XCH, (s.W - x0 + 15) & ~15);
    if (x0) __syncthreads();
    if (diff) {  // a token's 2 x 2 patch per 16 bytes
      const int nx = xc >> 1, np = 8 * HB * nx;
      const f32x4* src = diff + ((int64_t)f * s.C + c) * s.Hp * s.Wp;
      constexpr int U = 4;  // pieces a thread loads before it stores them
      for (int i0 = threadIdx.x; i0 < np; i0 += U * BAND_THREADS) {
        f32x4 d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * BAND_THREADS, hp = i / nx, wp = (x0 >> 1) + i - hp * nx;
          d[u] = hp < s.Hp && wp < s.Wp ? src[hp * s.Wp + wp] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * BAND_THREADS, hp = i / nx, xl = i - hp * nx;
          if (i >= np) continue;
          *(float2*)&sd[2 * hp][2 * xl] = make_float2(d[u][0], d[u][1]);
          *(float2*)&sd[2 * hp + 1][2 * xl] = make_float2(d[u][2], d[u][3]);
        }
      }
    } else {
      for (int i = threadIdx.x; i < 16 * HB * xc; i += BAND_THREADS) {
        const int h = i / xc, x = i - h * xc;
        sd[h][x] = h < s.H && x0 + x < s.W ? guided_diff(vL, vS, n, B, w, tok_offset(s, c, f, h, x0 + x)) : 0.0f;
      }
    }
    __syncthreads();
    if (live) {
      uint32_t m[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) m[i] = ((uint32_t)kw * (uint32_t)(x0 + 4 * g + i)) % W;
      for (int xk = 0; xk < xc; xk += 16) {
        float2 t[4];
        f32x4 a[HB];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          t[i] = twW[m[i]];
          m[i] = add_mod(m[i], step16, W);
        }
#pragma unroll
        for (int b = 0; b < HB; ++b) a[b] = *(const f32x4*)&sd[16 * b + jq][xk + 4 * g];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int b = 0; b < HB; ++b) {
            yr[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][i], t[i].x, yr[b], 0, 0, 0);
            yi[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][i], t[i].y, yi[b], 0, 0, 0);
          }
      }
    }
  }
  const double norm = (kw == 0 || 2 * kw == s.W ? 1.0 : 2.0) * inv_sum(1.0 / s.W, sumW);
  double acc[3] = {0.0, 0.0, 0.0};
  const double rH = 1.0 / s.H;
  for (int kh0 = 0; live && kh0 <= s.H / 2; kh0 += 16) {
    const uint32_t kh = kh0 + jq, steph = (16u * kh) % H;
    uint32_t m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = (kh * (uint32_t)(4 * g + r)) % H;
    f32x4 p = {0.0f, 0.0f, 0.0f, 0.0f}, q = p, u = p, v = p;  // sums of yr tx, yi ty, yr ty, yi tx
#pragma unroll
    for (int b = 0; b < HB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float2 t = twH[m[r]];
        m[r] = add_mod(m[r], steph, H);
        p = __builtin_amdgcn_mfma_f32_16x16x4f32(t.x, yr[b][r], p, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f32_16x16x4f32(t.y, yi[b][r], q, 0, 0, 0);
        u = __builtin_amdgcn_mfma_f32_16x16x4f32(t.y, yr[b][r], u, 0, 0, 0);
        v = __builtin_amdgcn_mfma_f32_16x16x4f32(t.x, yi[b][r], v, 0, 0, 0);
      }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = kh0 + 4 * g + r;
      if (k > s.H / 2 || kw > s.W / 2) continue;
      const double re = (double)(p[r] - q[r]), im = (double)(u[r] + v[r]);
      const double re2 = (double)(p[r] + q[r]), im2 = (double)(v[r] - u[r]);  // row H - k
      const double e = re * re + im * im, e2 = k == 0 || 2 * k == s.H ? 0.0 : re2 * re2 + im2 * im2;
      add_band(acc, spatial_band(k, kw, s.H, s.W), (e + e2) * (norm * inv_sum(rH, sumH[k])));
    }
  }
  block_sum3(acc[0], acc[1], acc[2], part + 3 * (int64_t)blockIdx.x);
}

// Block 0 of the temporal pass forms the sums of the rows' frequencies (W), block 1 those
// of the columns' (H), which the spatial pass divides by.
__device__ __forceinline__ void spatial_sums(const BandShape& s, float* __restrict__ dsum) {
  static_assert(BAND_MAX_H <= BAND_MAX_W, "one table's room");
  if (blockIdx.x == 0) freq_sums(dsum, s.W);
  else freq_sums(dsum + s.W / 2 + 1, s.H);
}

// Temporal block (patch_t 1: a frame's series are contiguous): 64 series a wave,
// lane jq the four from 4 jq on, "B" operands of four MFMAs as they are loaded.  With
// `diff` (patch 1 x 2 x 2) those four, one channel of one token, go there too.
__global__ __launch_bounds__(BAND_THREADS) void band_temporal_rows_kernel(BandShape s, int B, float w,
                                                                          const float* __restrict__ vL,
                                                                          const float* __restrict__ vS, int64_t n,
                                                                          f32x4* __restrict__ diff,
                                                                          float* __restrict__ dsum,
                                                                          double* __restrict__ part) {
  if (blockIdx.x < BAND_EXTRA) {
    spatial_sums(s, dsum);
    return;
  }
  __shared__ float2 tw[BAND_MAX_F];
  __shared__ float dev[BAND_MAX_F], sumF[BAND_MAX_F];
  fill_temporal(tw, dev, sumF, s.F);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int jq = lane & 15, g = lane >> 4;
  const int64_t total = (int64_t)s.Hp * s.Wp * s.P;  // series, a multiple of 4
  const int64_t i0 = ((int64_t)xcd_remap(blockIdx.x - BAND_EXTRA, gridDim.x - BAND_EXTRA) * 4 + wave) * 64 + 4 * jq;
  const bool in = i0 < total;
  const int64_t base = in ? i0 : 0;
  const uint32_t F = s.F;
  // the piece's place in frame 0, and the pieces of a frame
  const int64_t T = (int64_t)s.Hp * s.Wp, frame = s.C * T;
  const uint32_t b32 = (uint32_t)base, P = s.P;  // (a latent holds at most 2^31 values)
  f32x4* const dst = diff + (int64_t)(b32 % P / 4) * T + b32 / P;
  const double rF = 1.0 / s.F;
  double acc[3] = {0.0, 0.0, 0.0};
  for (int kf0 = 0; kf0 <= s.F / 2; kf0 += 16) {
    const uint32_t kf = kf0 + jq, step4 = (4u * kf) % F;
    uint32_t m = (kf * (uint32_t)g) % F;
    f32x4 re[4], im[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) re[i] = im[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int U = 3;  // steps of 4 frames whose loads are issued together
    for (int f0 = 0; f0 < s.F; f0 += 4 * U) {
      f32x4 d[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        d[u] = guided_diff4(vL, vS, n, B, w, (int64_t)min(f0 + 4 * u + g, s.F - 1) * total + base);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool live = in && f0 + 4 * u + g < s.F;
        if (live && diff && kf0 == 0) dst[(f0 + 4 * u + g) * frame] = d[u];
        const float2 t = tw[m];
        m = add_mod(m, step4, F);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = live ? d[u][i] : 0.0f;
          re[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.x, v, re[i], 0, 0, 0);
          im[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.y, v, im[i], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = kf0 + 4 * g + r;
      if (k > s.F / 2) continue;
      double e = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) e += (double)re[i][r] * re[i][r] + (double)im[i][r] * im[i][r];
      add_band(acc, axis_band(k, s.F), e * ((k == 0 || 2 * k == s.F ? 1.0 : 2.0) * inv_sum(rF, sumF[k])));
    }
  }
  block_sum3(acc[0], acc[1], acc[2], part + 3 * (int64_t)(blockIdx.x - BAND_EXTRA));
}

// Temporal energies of the other layouts (patch_t > 1, or velocities that are not
// 16-byte aligned).  One thread per (c, h, w) series, numbered in the token order of one frame
// group so that neighbouring threads read neighbouring floats.
__global__ __launch_bounds__(BAND_THREADS) void band_temporal_kernel(BandShape s, int B, float w,
                                                                    const float* __restrict__ vL,
                                                                    const float* __restrict__ vS, int64_t n,
                                                                    float* __restrict__ dsum,
                                                                    double* __restrict__ part) {
  if (blockIdx.x < BAND_EXTRA) {
    spatial_sums(s, dsum);
    return;
  }
  __shared__ float ser[BAND_MAX_F][BAND_THREADS];
  __shared__ float2 tw[BAND_MAX_F];
  __shared__ float dev[BAND_MAX_F], sumF[BAND_MAX_F];
  fill_temporal(tw, dev, sumF, s.F);
  const int64_t i = (int64_t)(blockIdx.x - BAND_EXTRA) * BAND_THREADS + threadIdx.x;
  const int Q = s.C * s.ph * s.pw;
  const int64_t total = (int64_t)s.Hp * s.Wp * Q;
  const bool live = i < total;
  int c = 0, h = 0, x = 0;
  if (live) {
    const int64_t lp = i / Q;
    const int e = (int)(i % Q);
    const int iw = e % s.pw, ih = (e / s.pw) % s.ph;
    c = e / (s.ph * s.pw);
    h = (int)(lp / s.Wp) * s.ph + ih;
    x = (int)(lp % s.Wp) * s.pw + iw;
    for (int f = 0; f < s.F; ++f) ser[f][threadIdx.x] = guided_diff(vL, vS, n, B, w, tok_offset(s, c, f, h, x));
  }
  __syncthreads();
  double acc[3] = {0.0, 0.0, 0.0};
  if (live) {
    const double rF = 1.0 / s.F;
    for (int kf = 0; kf < s.F; ++kf) {
      float re = 0.0f, im = 0.0f;
      int m = 0;  // kf * f mod F
      for (int f = 0; f < s.F; ++f) {
        const float d = ser[f][threadIdx.x];
        const float2 t = tw[m];
        re = fmaf(d, t.x, re);
        im = fmaf(d, t.y, im);
        m += kf;
        if (m >= s.F) m -= s.F;
      }
      const double e = ((double)re * re + (double)im * im) * inv_sum(rF, sumF[fold(kf, s.F)]);
      const int b = axis_band(kf, s.F);
      acc[0] += b == 0 ? e : 0.0;
      acc[1] += b == 1 ? e : 0.0;
      acc[2] += b == 2 ? e : 0.0;
    }
  }
  block_sum3(acc[0], acc[1], acc[2], part + 3 * (int64_t)(blockIdx.x - BAND_EXTRA));
}

// Sums the partials in a fixed order, one wave per quantity.  energy[0..2] spatial,
// [3..5] temporal.
// With step partials (pairs (sum d^2, sum p_L^2) of the calibration step
// kernel) it also writes score[b] = sqrt(energy[b]) / max(||p_L||, eps).
constexpr int BAND_FINISH_THREADS = 7 * 64;

__global__ __launch_bounds__(BAND_FINISH_THREADS) void band_finish_kernel(int ns, const double* __restrict__ part_s, int nt,
                                                          const double* __restrict__ part_t, int nstep,
                                                          const double* __restrict__ step_part, double eps,
                                                          double* __restrict__ energy,
                                                          double* __restrict__ score) {
  __shared__ double tot[7];
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double* p = q < 3 ? part_s + q : (q < 6 ? part_t + (q - 3) : step_part + 1);
  const int cnt = q < 3 ? ns : (q < 6 ? nt : (step_part ? nstep : 0));
  const int stride = q < 6 ? 3 : 2;
  double a = 0.0;
#pragma unroll 4
  for (int i = lane; i < cnt; i += 64) a += p[(int64_t)i * stride];
  a = wave_sum_d(a);
  if (lane == 0) tot[q] = a;
  __syncthreads();
  if (threadIdx.x < 6) {
    energy[threadIdx.x] = tot[threadIdx.x];
    if (step_part && score) {
      const double dn = sqrt(tot[6]);
      score[threadIdx.x] = sqrt(tot[threadIdx.x]) / (dn > eps ? dn : eps);
    }
  }
}

struct BandLayout {
  size_t diff, dsum, part_s, part_t, energy, total;
  int kwg, ns, nt;
};

// Layouts whose d goes through the workspace (where the velocities are aligned).
bool planar(const BandShape& s) { return s.pt == 1 && s.ph == 2 && s.pw == 2; }

BandLayout band_layout(const BandShape& s) {
  BandLayout b{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_256(off + bytes);
    return o;
  };
  b.kwg = s.W / 2 / BAND_COLS + 1;
  b.ns = b.kwg * s.C * s.F;
  b.nt = (int)(((int64_t)s.Hp * s.Wp * s.C * s.ph * s.pw + BAND_THREADS - 1) / BAND_THREADS);
  b.diff = take(planar(s) ? (size_t)s.C * s.F * s.H * s.W * sizeof(float) : 0);
  b.dsum = take((size_t)(s.W / 2 + s.H / 2 + 2) * sizeof(float));
  b.part_s = take((size_t)b.ns * 3 * 8);
  b.part_t = take((size_t)b.nt * 3 * 8);
  b.energy = take(6 * 8);
  b.total = off;
  return b;
}

BandShape make_shape(int C, int F, int H, int W, int pt, int ph, int pw) {
  BandShape s{C, F, H, W, pt, ph, pw, H / ph, W / pw, C * pt * ph * pw};
  return s;
}

}  // namespace

track_status band_check(int C, int F, int H, int W, int pt, int ph, int pw) {
  if (C < 1 || F < 1 || H < 1 || W < 1 || pt < 1 || ph < 1 || pw < 1)
    return fail(TRACK_E_SHAPE, "bands: bad latent %dx%dx%dx%d or patch %dx%dx%d", C, F, H, W, pt, ph, pw);
  if (F % pt || H % ph || W % pw) return fail(TRACK_E_SHAPE, "bands: latent not divisible by the patch");
  if (W > BAND_MAX_W || H > BAND_MAX_H || F > BAND_MAX_F)
    return fail(TRACK_E_UNSUPPORTED, "bands: supports W <= %d, H <= %d, F <= %d (got %d, %d, %d)", BAND_MAX_W,
                BAND_MAX_H, BAND_MAX_F, W, H, F);
  if ((int64_t)C * F * H * W > ((int64_t)1 << 31)) return fail(TRACK_E_UNSUPPORTED, "bands: latent too large");
  return TRACK_OK;
}

size_t band_workspace_bytes(int C, int F, int H, int W, int pt, int ph, int pw) {
  return band_layout(make_shape(C, F, H, W, pt, ph, pw)).total;
}

size_t band_energy_offset(int C, int F, int H, int W, int pt, int ph, int pw) {
  return band_layout(make_shape(C, F, H, W, pt, ph, pw)).energy;
}

track_status band_scores(int C, int F, int H, int W, int pt, int ph, int pw, int B, float w, const float* vel_L,
                         const float* vel_S, const double* step_partial, int64_t n_step_partials, double eps, void* ws,
                         double* energy_dev, double* score_dev, hipStream_t st) {
  {
    const track_status c = band_check(C, F, H, W, pt, ph, pw);
    if (c != TRACK_OK) return c;
  }
  if (B != 1 && B != 2) return fail(TRACK_E_INVALID, "bands: batch must be 1 or 2");
  if (!vel_L || !vel_S || !ws) return fail(TRACK_E_INVALID, "bands: null pointer");
  const BandShape s = make_shape(C, F, H, W, pt, ph, pw);
  const BandLayout L = band_layout(s);
  uint8_t* base = (uint8_t*)ws;
  float* dsum = (float*)(base + L.dsum);
  double* part_s = (double*)(base + L.part_s);
  double* part_t = (double*)(base + L.part_t);
  double* energy = energy_dev ? energy_dev : (double*)(base + L.energy);
  const int64_t n = (int64_t)C * F * H * W;  // floats per branch
  ProfScope prof(TRACK_PROF_STEP, st);
  const bool aligned = (((uintptr_t)vel_L | (uintptr_t)vel_S) & 15) == 0 && n % 4 == 0 && s.P % 4 == 0;
  f32x4* const diff = aligned && planar(s) ? (f32x4*)(base + L.diff) : nullptr;
  if (aligned && pt == 1)
    band_temporal_rows_kernel<<<L.nt + BAND_EXTRA, BAND_THREADS, 0, st>>>(s, B, w, vel_L, vel_S, n, diff, dsum, part_t);
  else
    band_temporal_kernel<<<L.nt + BAND_EXTRA, BAND_THREADS, 0, st>>>(s, B, w, vel_L, vel_S, n, dsum, part_t);
  TRACK_LAUNCH_CHECK();
#define TRACK_BAND(HB) \
  band_spatial_kernel<HB><<<L.ns, BAND_THREADS, 0, st>>>(s, B, w, vel_L, vel_S, n, diff, dsum, L.kwg, part_s)
  const int hb = (H + 15) / 16;
  if (hb <= 2) TRACK_BAND(2);
  else if (hb <= 4) TRACK_BAND(4);
  else if (hb <= 6) TRACK_BAND(6);
  else if (hb <= 8) TRACK_BAND(8);
  else TRACK_BAND(16);
#undef TRACK_BAND
  TRACK_LAUNCH_CHECK();
  band_finish_kernel<<<1, BAND_FINISH_THREADS, 0, st>>>(L.ns, part_s, L.nt, part_t, (int)n_step_partials, step_partial, eps,
                                                energy, score_dev);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

}  // namespace track
