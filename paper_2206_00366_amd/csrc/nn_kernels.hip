// Warm-start surrogate kernels for gfx950: 3x3 dilated convolutions as
// implicit GEMMs on MFMA (bf16 x bf16 -> fp32, v_mfma_f32_16x16x32_bf16),
// their backward passes, masked MSE, Adam, and the feature / target /
// initial-field kernels that connect the network to the lattice solver.
//
// Layouts: activations (B, H, W, C) channels-last, C a multiple of 16;
// weights (Cout, 3, 3, Cin); bf16 values are stored as raw uint16 bits.
// Tap (ky, kx) reads the input at (h + (ky-1) d, w + (kx-1) d), zero outside.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rmrt {
namespace nn {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
// the same in memory, where callers' tensors start at any element
typedef u32x4_t bf16x8_mem __attribute__((aligned(2)));
typedef u32x2_t bf16x4_mem __attribute__((aligned(2)));
typedef float4_t float4_mem __attribute__((aligned(4)));

// D += A B on 16 x 16 x 32: lane l supplies row l % 16 of A and column l % 16 of
// B for the eight k of its group l / 16, and receives D[4 (l / 16) + i][l % 16],
// i = 0..3.  (Which k a group's elements are does not matter as long as A and B
// agree.)
__device__ __forceinline__ float4_t mfma32(u32x4_t a, u32x4_t b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0,
                                                 0, 0);
}

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                           // round to nearest even
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float sigmoidf_(float y) { return 1.0f / (1.0f + __expf(-y)); }

enum { EPI_NONE = 0, EPI_SILU = 1, EPI_SILU_GRAD = 2 };

// A wave computes `tiles` runs of 16 consecutive pixels x all Cout channels:
// D[channel][pixel] = W[channel][k] X[k][pixel], so that a lane holds four
// consecutive channels of one pixel and stores 16 bytes of y and 8 of a.  k runs
// over a tap's 32 channels, or over two taps of 16.  The weights (at most 72
// registers) are read once per wave; the inputs are read straight from memory,
// 16 bytes a lane, nine times over from the L1 and L2.  Backward-data runs this
// kernel on weights flipped by k_flip.
// Bound by memory: at 16 x 64 x 128 pixels, 32 -> 32 channels, x, y and a are
// 34 MB; 32 us with one tile per wave, 16-wide k and 2- and 4-byte stores (every
// wave read all weights for 16 pixels), 16 us now.
template <int CIN, int COUT>
__global__ void __launch_bounds__(256, 2)
    k_conv(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w, const float* __restrict__ bias,
           float* __restrict__ y_pre, uint16_t* __restrict__ a_out, const float* __restrict__ aux, int B, int H,
           int W, int dil, int epi, int tiles) {
  constexpr int NB = COUT / 16, S = CIN == 32 ? 9 : 5;
  const int lane = threadIdx.x & 63, m = lane & 15, kg = lane >> 4;
  const long wave = (long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const long P = (long)B * H * W;
  if (wave * tiles * 16 >= P) return;
  // tap and first channel of this lane's k group in step s
  auto tap_of = [&](int s) { return CIN == 32 ? s : 2 * s + (kg >> 1); };
  const int ch = CIN == 32 ? 8 * kg : 8 * (kg & 1);
  u32x4_t wf[NB][S];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int tap = tap_of(s);
      wf[nb][s] = u32x4_t{0u, 0u, 0u, 0u};
      if (CIN == 32 || tap < 9) wf[nb][s] = *(const bf16x8_mem*)(w + ((long)(nb * 16 + m) * 9 + tap) * CIN + ch);
    }
  float4_t bv[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
    bv[nb] = bias ? *(const float4_mem*)(bias + nb * 16 + 4 * kg) : float4_t{0.f, 0.f, 0.f, 0.f};
  for (int t = 0; t < tiles; ++t) {
    const long p0 = (wave * tiles + t) * 16;
    if (p0 >= P) return;
    const long p = p0 + m;
    long row;
    int wq;
    if (P <= 0x7fffffffL) {   // 32-bit divisions where they reach
      row = (uint32_t)p / (uint32_t)W;
      wq = (int)((uint32_t)p - (uint32_t)row * (uint32_t)W);
    } else {
      row = p / W;
      wq = (int)(p - row * W);
    }
    const int h = P <= 0x7fffffffL ? (int)((uint32_t)row % (uint32_t)H) : (int)(row % H);
    const bool ok = p < P;
    const uint16_t* xc = x + p * CIN + ch;
    u32x4_t xf[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int tap = tap_of(s), dy = tap / 3 - 1, dx = tap - 3 * (tap / 3) - 1;
      const long hh = (long)h + (long)dy * dil, ww = (long)wq + (long)dx * dil;
      const bool in = ok && tap < 9 && hh >= 0 && hh < H && ww >= 0 && ww < W;
      xf[s] = u32x4_t{0u, 0u, 0u, 0u};
      if (in) xf[s] = *(const bf16x8_mem*)(xc + ((long)dy * W + dx) * dil * CIN);
    }
    float4_t acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma32(wf[nb][s], xf[s], acc[nb]);
    if (!ok) continue;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const long o = p * COUT + nb * 16 + 4 * kg;
      float4_t v = acc[nb] + bv[nb];
      if (y_pre) *(float4_mem*)(y_pre + o) = v;
      if (epi == EPI_SILU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = v[i] * sigmoidf_(v[i]);
      } else if (epi == EPI_SILU_GRAD) {
        const float4_t yv = *(const float4_mem*)(aux + o);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float sg = sigmoidf_(yv[i]);
          v[i] = v[i] * sg * (1.f + yv[i] * (1.f - sg));
        }
      }
      if (a_out)
        *(bf16x4_mem*)(a_out + o) = u32x2_t{(uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                                         (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16)};
    }
  }
}

// wt[ci][ky][kx][co] = w[co][2 - ky][2 - kx][ci]: backward-data as a forward conv
__global__ void k_flip(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, int Cout, int Cin) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = Cout * 9 * Cin;
  if (i >= n) return;
  const int co = i / (9 * Cin);
  const int r = i - co * 9 * Cin;
  const int tap = r / Cin, ci = r - tap * Cin;
  const int ky = tap / 3, kx = tap % 3;
  wt[((long)ci * 9 + (2 - ky) * 3 + (2 - kx)) * Cout + co] = w[i];
}

// dW[co][tap][ci] = sum_p dY[p][co] X[p + tap][ci] and db[co] = sum_p dY[p][co].
// A workgroup takes a run of row segments of up to kSeg pixels.  Each segment's
// dY and the X windows of its nine taps go through LDS as words of two
// neighbouring pixels of one channel, so that a lane collects the eight pixels
// of its channel with four 4-byte reads (k = pixels, four groups of 16 lanes on
// consecutive pixel pairs: no bank conflicts).  Wave w takes the 16 x 16 block
// w % (MB NB) of the channel pairs for all taps and, where there are fewer blocks than
// waves, every KS-th run of 32 pixels.  An even dilation up to 32 shares one
// X window per tap row, others take one window per tap.
// Bound by LDS reads (40 a wave for 10 products) and the latency of one segment's
// loads; at 16 x 64 x 128 pixels, 32 x 32 channels: 129 us with 2-byte gathers
// from memory, one wave per tap and chunk, + 35 us for the sum of its partials
// and + 213 us for db (its last sum was one thread per channel), 16 + 5 us now
// together.
// Rows of up to kNarrow pixels (FLAT) would leave most of a segment empty:
// there a segment is kSeg consecutive pixels of the whole batch, whatever rows
// and images they lie in, with one window per tap.  131072 pixels in rows of W,
// 32 x 32 channels, dilation 1 / 2, by rows and flat (us, sums included): W = 1
// 1206 / 753 and 25 / 25, 8 173 / 114 and 26 / 27, 32 50 / 34 and 26 / 26, 64
// 34 / 25 and 25 / 25 (16 -> 16 channels 27 / 22 and 23 / 23: by rows).
constexpr int kSeg = 128, kWgBlocks = 512, kNarrow = 32;
inline long wgrad_items(int B, int H, int W) {
  return W <= kNarrow ? ((long)B * H * W + kSeg - 1) / kSeg : (long)B * H * ((W + kSeg - 1) / kSeg);
}
__host__ __device__ inline bool wgrad_shared_window(int dil) { return dil > 0 && dil % 2 == 0 && dil <= 32; }
__host__ __device__ inline int wgrad_window_pixels(int dil) {   // X pixels in LDS, a multiple of 2
  return wgrad_shared_window(dil) ? 3 * (kSeg + 2 * dil) : 9 * kSeg;
}
template <int CIN, int COUT>
struct WgradSplit {
  static constexpr int MB = COUT / 16, NB = CIN / 16, KS = 4 / (MB * NB);
};
template <int CIN, int COUT, bool FLAT>
__global__ void __launch_bounds__(256, 2)
    k_wgrad(const uint16_t* __restrict__ x, const uint16_t* __restrict__ dy, float* __restrict__ part,
            float* __restrict__ partb, int B, int H, int W, int dil, long items, long per_block) {
  constexpr int MB = WgradSplit<CIN, COUT>::MB, NB = WgradSplit<CIN, COUT>::NB, KS = WgradSplit<CIN, COUT>::KS;
  extern __shared__ __align__(16) uint32_t sh[];
  uint32_t* const shy = sh;                          // [kSeg / 2][COUT]
  uint32_t* const shx = sh + kSeg / 2 * COUT;        // [window pixels / 2][CIN]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 15, g = lane >> 4;
  const int blk = wave % (MB * NB), ks = wave / (MB * NB), a = blk / NB, c = blk % NB;
  const bool shared = !FLAT && wgrad_shared_window(dil);
  const int win = shared ? kSeg + 2 * dil : kSeg;    // pixels of a window
  const int nwin = shared ? 3 : 9;
  const int nseg = (W + kSeg - 1) / kSeg;
  const long P = (long)B * H * W;
  float4_t acc[9], accb = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
  // two pixels' eight channels (16 bytes each) as eight words of a pixel pair
  auto put = [](uint32_t* to, u32x4_t lo, u32x4_t hi) {
    u32x4_t r0, r1;
    r0[0] = (lo[0] & 0xffffu) | (hi[0] << 16);
    r0[1] = (lo[0] >> 16) | (hi[0] & 0xffff0000u);
    r0[2] = (lo[1] & 0xffffu) | (hi[1] << 16);
    r0[3] = (lo[1] >> 16) | (hi[1] & 0xffff0000u);
    r1[0] = (lo[2] & 0xffffu) | (hi[2] << 16);
    r1[1] = (lo[2] >> 16) | (hi[2] & 0xffff0000u);
    r1[2] = (lo[3] & 0xffffu) | (hi[3] << 16);
    r1[3] = (lo[3] >> 16) | (hi[3] & 0xffff0000u);
    *(u32x4_t*)to = r0;
    *(u32x4_t*)(to + 4) = r1;
  };
  const u32x4_t zero = u32x4_t{0u, 0u, 0u, 0u};
  const u32x4_t ones = u32x4_t{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  long it = (long)blockIdx.x * per_block;
  const long end = it + per_block < items ? it + per_block : items;
  for (; it < end; ++it) {
    const long row = FLAT ? 0 : it / nseg;           // b H + h
    const int w0 = FLAT ? 0 : (int)(it - row * nseg) * kSeg;
    const int h = FLAT ? 0 : (int)(row % H);
    const long p0 = FLAT ? it * kSeg : row * W + w0; // first pixel
    const long left = FLAT ? P - p0 : (long)W - w0;
    const int len = left < kSeg ? (int)left : kSeg;
    __syncthreads();                                 // the previous segment has been read
    for (int i = threadIdx.x; i < kSeg / 2 * (COUT / 8); i += 256) {
      const int pr = i / (COUT / 8), q = i % (COUT / 8);
      const uint16_t* src = dy + (p0 + 2 * pr) * COUT + 8 * q;
      const u32x4_t lo = 2 * pr < len ? *(const bf16x8_mem*)src : zero;
      const u32x4_t hi = 2 * pr + 1 < len ? *(const bf16x8_mem*)(src + COUT) : zero;
      put(shy + pr * COUT + 8 * q, lo, hi);
    }
    if constexpr (FLAT) {
      for (int i = threadIdx.x; i < kSeg / 2 * (CIN / 8); i += 256) {
        const int pr = i / (CIN / 8), q = i % (CIN / 8);
        const long p = p0 + 2 * pr, r0 = p / W, r1 = (p + 1) / W;
        const long h0 = r0 % H, h1 = r1 % H, x0 = p - r0 * W, x1 = p + 1 - r1 * W;
        const bool ok0 = 2 * pr < len, ok1 = 2 * pr + 1 < len;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
          const long ty = (long)(t / 3 - 1) * dil, tx = (long)(t % 3 - 1) * dil;
          const uint16_t* src = x + (p + ty * W + tx) * CIN + 8 * q;
          const bool in0 = ok0 && h0 + ty >= 0 && h0 + ty < H && x0 + tx >= 0 && x0 + tx < W;
          const bool in1 = ok1 && h1 + ty >= 0 && h1 + ty < H && x1 + tx >= 0 && x1 + tx < W;
          const u32x4_t lo = in0 ? *(const bf16x8_mem*)src : zero;
          const u32x4_t hi = in1 ? *(const bf16x8_mem*)(src + CIN) : zero;
          put(shx + (t * (kSeg / 2) + pr) * CIN + 8 * q, lo, hi);
        }
      }
    } else
    for (int i = threadIdx.x; i < nwin * (win / 2) * (CIN / 8); i += 256) {
      const int q = i % (CIN / 8), r = i / (CIN / 8), wi = r / (win / 2), pr = r - wi * (win / 2);
      const int ky = shared ? wi : wi / 3;
      const long hh = (long)h + (long)(ky - 1) * dil;
      const long ww = (long)w0 + (shared ? -(long)dil : (long)(wi - 3 * ky - 1) * dil) + 2 * pr;
      const uint16_t* src = x + ((row + (long)(ky - 1) * dil) * W + ww) * CIN + 8 * q;
      const bool in = hh >= 0 && hh < H;
      const u32x4_t lo = in && ww >= 0 && ww < W ? *(const bf16x8_mem*)src : zero;
      const u32x4_t hi = in && ww + 1 >= 0 && ww + 1 < W ? *(const bf16x8_mem*)(src + CIN) : zero;
      put(shx + r * CIN + 8 * q, lo, hi);
    }
    __syncthreads();
    for (int c0 = 16 * ks; 2 * c0 < len; c0 += 16 * KS) {   // pixel pairs c0 .. c0 + 15
      u32x4_t av;
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = shy[(c0 + 4 * i + g) * COUT + a * 16 + m];
      if (c == 0) accb = mfma32(av, ones, accb);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int base = (shared ? (t / 3) * (win / 2) + (t % 3) * (dil / 2) : t * (kSeg / 2)) + c0;
        u32x4_t bv;
#pragma unroll
        for (int i = 0; i < 4; ++i) bv[i] = shx[(base + 4 * i + g) * CIN + c * 16 + m];
        if (2 * c0 + 32 > len)   // pixels beyond the row: no product, whatever X holds there
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int px = 2 * (c0 + 4 * i + g);
            bv[i] &= px + 1 < len ? ~0u : px < len ? 0xffffu : 0u;
          }
        acc[t] = mfma32(av, bv, acc[t]);
      }
    }
  }
  // D[row = co][col = ci]: lane holds rows 4 g + i, column m
  const long slot = (long)blockIdx.x * KS + ks;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      part[((slot * COUT + a * 16 + 4 * g + i) * 9 + t) * CIN + c * 16 + m] = acc[t][i];
  if (c == 0 && m == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i) partb[slot * COUT + a * 16 + 4 * g + i] = accb[i];
}

// Sums of n partials of `len` floats (out) and `lenb` floats (outb, may be
// null): 32 neighbouring outputs (a whole line of each partial) and 32
// interleaved runs of partials per workgroup, then a tree over the runs: a fixed
// order.  Bound by latency and the read of the partials (19 MB for 32 x 32
// channels: 7.9 us with 16 outputs and 16 runs per workgroup, 4.8 now).
constexpr int kSumOuts = 32, kSumRuns = 32;
__global__ void __launch_bounds__(kSumOuts* kSumRuns)
    k_sum_partials(const float* __restrict__ part, float* __restrict__ out, int len, const float* __restrict__ partb,
                   float* __restrict__ outb, int lenb, int n) {
  __shared__ float sh[kSumRuns][kSumOuts + 1];
  const int e = threadIdx.x % kSumOuts, r = threadIdx.x / kSumOuts;
  const int nb = (len + kSumOuts - 1) / kSumOuts;
  const bool second = (int)blockIdx.x >= nb;
  const float* src = second ? partb : part;
  float* dst = second ? outb : out;
  const int l = second ? lenb : len;
  const int o = ((int)blockIdx.x - (second ? nb : 0)) * kSumOuts + e;
  float s = 0.f;
  if (o < l)
#pragma unroll 8
    for (int k = r; k < n; k += kSumRuns) s += src[(long)k * l + o];
  sh[r][e] = s;
  __syncthreads();
  for (int d = kSumRuns / 2; d > 0; d >>= 1) {
    if (r < d) sh[r][e] += sh[r + d][e];
    __syncthreads();
  }
  if (r == 0 && o < l) dst[o] = sh[0][e];
}

// sum of a double per thread over a 256-thread workgroup, valid in thread 0
__device__ __forceinline__ double block_sum(double s) {
  __shared__ double sh[4];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

// sum of the pixel weights: per-workgroup partials, which every workgroup of
// k_mse sums for itself (in one order)
__global__ void __launch_bounds__(256) k_wsum(const float* __restrict__ mask, long P, double* __restrict__ part) {
  double s = 0.0;
  for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < P; p += (long)gridDim.x * blockDim.x) s += mask[p];
  s = block_sum(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// masked MSE over the first C channels of out (stride Cs): per-workgroup loss
// partials; dout (bf16, stride Cs, zero in the padding channels).  Bound by
// latency (three short kernels, serial sums by one thread before: 72 us, now
// 12 us together at 16 x 64 x 128 pixels).
__global__ void __launch_bounds__(256)
    k_mse(const float* __restrict__ out, int Cs, const float* __restrict__ tgt, const float* __restrict__ mask, long P,
          int C, const double* __restrict__ wpart, int nw, float* __restrict__ inv_den_p, uint16_t* __restrict__ dout,
          double* __restrict__ part) {
  double ws = 0.0;
  for (int k = threadIdx.x; k < nw; k += 256) ws += wpart[k];
  ws = block_sum(ws);
  const float inv_den = ws > 0.0 ? (float)(1.0 / ws) : 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) inv_den_p[0] = inv_den;
  double s = 0.0;
  for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < P; p += (long)gridDim.x * blockDim.x) {
    const float mk = mask[p];
    auto grad = [&](int c) {
      const float dlt = out[p * Cs + c] - tgt[p * C + c];
      s += (double)mk * dlt * dlt;
      return (uint32_t)f2bf(2.f * mk * dlt * inv_den);
    };
    if (Cs % 8 == 0) {
      for (int c0 = 0; c0 < Cs; c0 += 8) {
        u32x4_t v = u32x4_t{0u, 0u, 0u, 0u};
        if (c0 < C) {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (c0 + i < C) v[i / 2] |= grad(c0 + i) << (16 * (i & 1));
        }
        *(bf16x8_mem*)(dout + p * Cs + c0) = v;
      }
    } else {
      for (int c = 0; c < Cs; ++c) dout[p * Cs + c] = c < C ? (uint16_t)grad(c) : (uint16_t)0;
    }
  }
  s = block_sum(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}
__global__ void __launch_bounds__(256) k_sum_final(const double* __restrict__ part, int nb, const float* __restrict__ scale,
                                                   double* __restrict__ out) {
  double s = 0.0;
  for (int k = threadIdx.x; k < nb; k += 256) s += part[k];
  s = block_sum(s);
  if (threadIdx.x == 0) out[0] = s * (double)scale[0];
}

// Adam with bias correction; w32 master weights, optional bf16 copy
__global__ void k_adam(float* __restrict__ w, uint16_t* __restrict__ wbf, const float* __restrict__ g,
                       float* __restrict__ mo, float* __restrict__ vo, long n, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float m = b1 * mo[i] + (1.f - b1) * gi;
  const float v = b2 * vo[i] + (1.f - b2) * gi * gi;
  mo[i] = m;
  vo[i] = v;
  const float wi = w[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
  w[i] = wi;
  if (wbf) wbf[i] = f2bf(wi);
}

__global__ void k_to_bf16(const float* __restrict__ src, uint16_t* __restrict__ dst, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = f2bf(src[i]);
}

// ---------------------------------------------------------------------------
// Glue between the lattice solver (fine grid, nodes x-fastest, walls at the
// y faces) and the network (coarse grid, k x k blocks, channels-last).
// Coarse pixel (b, i, j): rows i (y), columns j (x).  The Poiseuille prior is
// 4 y (H - y) / H^2 at the physical height y of the cell centre.
// ---------------------------------------------------------------------------
// colfrac[b][x] = solid fraction of column x; gfrac[b] = solid fraction of sample b.
// Bound by latency: 64 columns and 16 interleaved runs of rows per workgroup (16
// samples of 512 x 256: one thread per column and per sample before, 98 + 38 us,
// now 5 + 3 us).
__global__ void __launch_bounds__(1024)
    k_colfrac(const uint8_t* __restrict__ solid, int B, int nx, int ny, float* __restrict__ colfrac) {
  __shared__ int sh[16][64];
  const int e = threadIdx.x & 63, r = threadIdx.x >> 6;
  const int per = (nx + 63) / 64, b = blockIdx.x / per, x = (blockIdx.x % per) * 64 + e;
  int cnt = 0;
  if (x < nx)
#pragma unroll 4
    for (int y = r; y < ny; y += 16) cnt += solid[((long)b * ny + y) * nx + x] ? 1 : 0;
  sh[r][e] = cnt;
  __syncthreads();
  if (r == 0 && x < nx) {
    for (int k = 1; k < 16; ++k) cnt += sh[k][e];
    colfrac[(long)b * nx + x] = (float)cnt / (float)ny;
  }
}
__global__ void __launch_bounds__(256) k_gfrac(const float* __restrict__ colfrac, int nx, float* __restrict__ gfrac) {
  double s = 0.0;
  for (int x = threadIdx.x; x < nx; x += 256) s += colfrac[(long)blockIdx.x * nx + x];
  s = block_sum(s);
  if (threadIdx.x == 0) gfrac[blockIdx.x] = (float)(s / nx);
}

// features: ch0 = solid fraction of the block, ch1 = prior, ch2 = Re / re_scale,
// ch3 = solid fraction of the block's columns over the full height (local
// constriction), ch4 = solid fraction of the whole channel, ch5.. = 0
__global__ void k_features(const uint8_t* __restrict__ solid, const float* __restrict__ re, int B, int nx, int ny, int k,
                           float dy, float re_scale, const float* __restrict__ colfrac, const float* __restrict__ gfrac,
                           uint16_t* __restrict__ x0, int Cs) {
  const int hc = ny / k, wc = nx / k;
  const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (long)B * hc * wc) return;
  const int b = (int)(p / ((long)hc * wc));
  const int r = (int)(p - (long)b * hc * wc);
  const int i = r / wc, j = r - i * wc;
  int cnt = 0;
  for (int a = 0; a < k; ++a)
    for (int c = 0; c < k; ++c) cnt += solid[(long)b * nx * ny + (long)(i * k + a) * nx + (j * k + c)] ? 1 : 0;
  const float Hh = ny * dy;
  const float y = (i * k + 0.5f * k) * dy;
  const float prior = 4.f * y * (Hh - y) / (Hh * Hh);
  float col = 0.f;
  for (int c = 0; c < k; ++c) col += colfrac[(long)b * nx + j * k + c];
  col /= (float)k;
  for (int c = 0; c < Cs; ++c) {
    float v = 0.f;
    if (c == 0) v = (float)cnt / (float)(k * k);
    if (c == 1) v = prior;
    if (c == 2) v = re[b] / re_scale;
    if (c == 3) v = col;
    if (c == 4) v = gfrac[b];
    x0[p * Cs + c] = f2bf(v);
  }
}

// targets: fluid means over the block of (u / Ut - prior(y_node)), v / Ut,
// (rho - 1) rho_scale; weight = fluid fraction of the block
__global__ void k_targets(const double* __restrict__ rho, const double* __restrict__ u, const uint8_t* __restrict__ solid,
                          int B, int nx, int ny, int k, float dy, float Ut, float rho_scale, float* __restrict__ tgt,
                          float* __restrict__ wgt) {
  const int hc = ny / k, wc = nx / k;
  const long p = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (long)B * hc * wc) return;
  const int b = (int)(p / ((long)hc * wc));
  const int r = (int)(p - (long)b * hc * wc);
  const int i = r / wc, j = r - i * wc;
  const long N = (long)nx * ny;
  const float Hh = ny * dy;
  double s0 = 0, s1 = 0, s2 = 0;
  int cnt = 0;
  for (int a = 0; a < k; ++a)
    for (int c = 0; c < k; ++c) {
      const int yy = i * k + a, xx = j * k + c;
      const long n = (long)yy * nx + xx;
      if (solid[b * N + n]) continue;
      const float y = (yy + 0.5f) * dy;
      const float prior = 4.f * y * (Hh - y) / (Hh * Hh);
      s0 += u[(long)b * 2 * N + n] / Ut - prior;
      s1 += u[(long)b * 2 * N + N + n] / Ut;
      s2 += (rho[b * N + n] - 1.0) * rho_scale;
      ++cnt;
    }
  const double inv = cnt ? 1.0 / cnt : 0.0;
  tgt[p * 3 + 0] = (float)(s0 * inv);
  tgt[p * 3 + 1] = (float)(s1 * inv);
  tgt[p * 3 + 2] = (float)(s2 * inv);
  wgt[p] = (float)cnt / (float)(k * k);
}

// initial fields on the fine grid from the coarse prediction (bilinear,
// positions (node + 1/2) / k - 1/2 in coarse units, clamped):
// u = Ut (prior(y) + o0), v = Ut o1, rho = 1 + o2 / rho_scale; zero velocity in solids
__global__ void k_warm_fields(const float* __restrict__ out, int Cs, int B, int nx, int ny, int k, float dy, float Ut,
                              float rho_scale, const uint8_t* __restrict__ solid, double* __restrict__ rho,
                              double* __restrict__ u) {
  const int hc = ny / k, wc = nx / k;
  const long N = (long)nx * ny;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)B * N) return;
  const int b = (int)(t / N);
  const long n = t - (long)b * N;
  const int yy = (int)(n / nx), xx = (int)(n - (long)yy * nx);
  float py = (yy + 0.5f) / k - 0.5f, px = (xx + 0.5f) / k - 0.5f;
  py = fminf(fmaxf(py, 0.f), (float)(hc - 1));
  px = fminf(fmaxf(px, 0.f), (float)(wc - 1));
  const int i0 = (int)floorf(py), j0 = (int)floorf(px);
  const int i1 = min(i0 + 1, hc - 1), j1 = min(j0 + 1, wc - 1);
  const float fy = py - i0, fx = px - j0;
  float o[3];
  for (int c = 0; c < 3; ++c) {
    const float* base = out + (long)b * hc * wc * Cs;
    const float v00 = base[((long)i0 * wc + j0) * Cs + c], v01 = base[((long)i0 * wc + j1) * Cs + c];
    const float v10 = base[((long)i1 * wc + j0) * Cs + c], v11 = base[((long)i1 * wc + j1) * Cs + c];
    o[c] = (v00 * (1 - fx) + v01 * fx) * (1 - fy) + (v10 * (1 - fx) + v11 * fx) * fy;
  }
  const float Hh = ny * dy;
  const float y = (yy + 0.5f) * dy;
  const float prior = 4.f * y * (Hh - y) / (Hh * Hh);
  const bool s = solid && solid[b * N + n];
  rho[b * N + n] = 1.0 + (double)o[2] / rho_scale;
  u[(long)b * 2 * N + n] = s ? 0.0 : (double)(Ut * (prior + o[0]));
  u[(long)b * 2 * N + N + n] = s ? 0.0 : (double)(Ut * o[1]);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
hipError_t launch_conv(const uint16_t* x, const uint16_t* w, const float* bias, float* y_pre, uint16_t* a_out,
                       const float* aux, int B, int H, int W, int Cin, int Cout, int dil, int epi, hipStream_t s) {
  const long P = (long)B * H * W;
  const long runs = (P + 15) / 16;
  // more pixels per wave once the chip has two waves per SIMD
  const int tiles = (int)(runs / 2048 < 1 ? 1 : runs / 2048 > 8 ? 8 : runs / 2048);
  const unsigned blocks = (unsigned)(((runs + tiles - 1) / tiles + 3) / 4);
#define CONV_CASE(CI, CO)                                                                                      \
  if (Cin == CI && Cout == CO) {                                                                               \
    hipLaunchKernelGGL((k_conv<CI, CO>), dim3(blocks), dim3(256), 0, s, x, w, bias, y_pre, a_out, aux, B, H, W, \
                       dil, epi, tiles);                                                                       \
    return hipGetLastError();                                                                                  \
  }
  CONV_CASE(16, 16) CONV_CASE(16, 32) CONV_CASE(32, 16) CONV_CASE(32, 32)
#undef CONV_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_flip(const uint16_t* w, uint16_t* wt, int Cout, int Cin, hipStream_t s) {
  const int n = Cout * 9 * Cin;
  hipLaunchKernelGGL(k_flip, dim3((n + 255) / 256), dim3(256), 0, s, w, wt, Cout, Cin);
  return hipGetLastError();
}

// Workgroups of k_wgrad (row segments shared evenly) and their partial sums.
static long wgrad_blocks(int B, int H, int W, long* per_block) {
  const long items = wgrad_items(B, H, W);
  *per_block = (items + kWgBlocks - 1) / kWgBlocks;
  return (items + *per_block - 1) / *per_block;
}
static size_t wgrad_partial_floats(long blocks, int Cin, int Cout) {
  return (size_t)blocks * (4 / ((Cin / 16) * (Cout / 16))) * ((size_t)9 * Cin * Cout + Cout);
}
// Scratch of a launch, and scratch for these sizes and all smaller ones (an even
// share can need fewer workgroups for more segments: 257 for 513, 512 for 512).
size_t wgrad_need_floats(int B, int H, int W, int Cin, int Cout) {
  long per = 0;
  return wgrad_partial_floats(wgrad_blocks(B, H, W, &per), Cin, Cout);
}
size_t wgrad_scratch_floats(int B, int H, int W, int Cin, int Cout) {
  const long items = wgrad_items(B, H, W);
  return wgrad_partial_floats(items < kWgBlocks ? items : kWgBlocks, Cin, Cout);
}

hipError_t launch_wgrad(const uint16_t* x, const uint16_t* dy, int B, int H, int W, int Cin, int Cout, int dil, float* dw,
                        float* db, float* part, size_t part_floats, hipStream_t s) {
  const long items = wgrad_items(B, H, W);
  const bool flat = W <= kNarrow;
  long per = 0;
  const long blocks = wgrad_blocks(B, H, W, &per);
  if (wgrad_partial_floats(blocks, Cin, Cout) > part_floats) return hipErrorInvalidValue;
  const int slots = (int)blocks * (4 / ((Cin / 16) * (Cout / 16)));
  const int len = 9 * Cin * Cout;
  float* partb = part + (size_t)slots * len;
  const size_t lds = ((size_t)kSeg / 2 * Cout + (size_t)(flat ? 9 * kSeg : wgrad_window_pixels(dil)) / 2 * Cin) * 4;
#define WG_CASE(CI, CO)                                                                                             \
  if (Cin == CI && Cout == CO) {                                                                                    \
    if (flat)                                                                                                       \
      hipLaunchKernelGGL((k_wgrad<CI, CO, true>), dim3((unsigned)blocks), dim3(256), lds, s, x, dy, part, partb, B, H, W, \
                         dil, items, per);                                                                          \
    else                                                                                                            \
      hipLaunchKernelGGL((k_wgrad<CI, CO, false>), dim3((unsigned)blocks), dim3(256), lds, s, x, dy, part, partb, B, H, W, \
                         dil, items, per);                                                                          \
  } else
  WG_CASE(16, 16) WG_CASE(16, 32) WG_CASE(32, 16) WG_CASE(32, 32) { return hipErrorInvalidValue; }
#undef WG_CASE
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int lenb = db ? Cout : 0;
  const int groups = (len + kSumOuts - 1) / kSumOuts + (lenb + kSumOuts - 1) / kSumOuts;
  hipLaunchKernelGGL(k_sum_partials, dim3((unsigned)groups), dim3(kSumOuts * kSumRuns), 0, s, part, dw, len, partb, db,
                     lenb, slots);
  return hipGetLastError();
}

// scratch: >= 2 * kMseBlocks doubles; loss: one double (device); inv_den: one float (device)
constexpr int kMseBlocks = 512;
hipError_t launch_mse(const float* out, int Cs, const float* tgt, const float* mask, long P, int C, uint16_t* dout,
                      double* scratch, float* inv_den, double* loss, hipStream_t s) {
  const int nb = kMseBlocks;
  hipLaunchKernelGGL(k_wsum, dim3(nb), dim3(256), 0, s, mask, P, scratch);
  hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, out, Cs, tgt, mask, P, C, scratch, nb, inv_den, dout,
                     scratch + nb);
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, scratch + nb, nb, inv_den, loss);
  return hipGetLastError();
}

hipError_t launch_adam(float* w, uint16_t* wbf, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
                       float eps, float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, wbf, g, m, v, n, lr, b1, b2, eps,
                     c1, c2);
  return hipGetLastError();
}

hipError_t launch_to_bf16(const float* src, uint16_t* dst, long n, hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
  return hipGetLastError();
}

// scratch: B * (nx + 1) floats
hipError_t launch_features(const uint8_t* solid, const float* re, int B, int nx, int ny, int k, float dy, float re_scale,
                           uint16_t* x0, int Cs, float* scratch, hipStream_t s) {
  const long P = (long)B * (ny / k) * (nx / k);
  float* colfrac = scratch;
  float* gfrac = scratch + (long)B * nx;
  hipLaunchKernelGGL(k_colfrac, dim3((unsigned)((long)B * ((nx + 63) / 64))), dim3(1024), 0, s, solid, B, nx, ny, colfrac);
  hipLaunchKernelGGL(k_gfrac, dim3(B), dim3(256), 0, s, colfrac, nx, gfrac);
  hipLaunchKernelGGL(k_features, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, solid, re, B, nx, ny, k, dy,
                     re_scale, colfrac, gfrac, x0, Cs);
  return hipGetLastError();
}

hipError_t launch_targets(const double* rho, const double* u, const uint8_t* solid, int B, int nx, int ny, int k,
                          float dy, float Ut, float rho_scale, float* tgt, float* wgt, hipStream_t s) {
  const long P = (long)B * (ny / k) * (nx / k);
  hipLaunchKernelGGL(k_targets, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, rho, u, solid, B, nx, ny, k, dy,
                     Ut, rho_scale, tgt, wgt);
  return hipGetLastError();
}

hipError_t launch_warm_fields(const float* out, int Cs, int B, int nx, int ny, int k, float dy, float Ut,
                              float rho_scale, const uint8_t* solid, double* rho, double* u, hipStream_t s) {
  const long n = (long)B * nx * ny;
  hipLaunchKernelGGL(k_warm_fields, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, Cs, B, nx, ny, k, dy, Ut,
                     rho_scale, solid, rho, u);
  return hipGetLastError();
}

}  // namespace nn
}  // namespace rmrt
