// Non-MFMA kernels: 1x1 convolutions with few outputs (e.g. a 1-channel head),
// depthwise 3x3, ReLU
// backward, bias gradient, max-pool, upsample-concat, MSE and gradient
// accumulation.  All reductions run in a fixed order (per-thread serial sums,
// fixed LDS trees, fixed split order), so results are bit-reproducible.
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace tgpk {

bool mfma_fwd_ok(int dt, const ConvShape& s);
bool mfma_wgrad_ok(int dt, const ConvShape& s);
bool conv_dgrad_tile_now(const ConvShape& t, int n);
hipError_t conv_dgrad_tile(int n, const void* const* dz, const void* w, void* const* dx,
                           const ConvShape& t, float* const* part, size_t part_cap,
                           hipStream_t st);
hipError_t conv_forward_mfma(const void* x, const void* w, const float* b, void* y,
                             const ConvShape& s, int relu, float* part, size_t part_cap,
                             hipStream_t st);
size_t wgrad_mfma_partial_floats(const ConvShape& s);
hipError_t conv_wgrad_mfma(const void* x, const void* dz, float* dw, float* partial,
                           const ConvShape& s, hipStream_t st, ReduceJob* defer);
hipError_t conv_forward_mfma_n(int n, const void* const* x, const void* w, const float* b,
                               void* const* y, const ConvShape& s, int relu, float* const* part,
                               size_t part_cap, hipStream_t st);
hipError_t conv_wgrad_mfma_n(int n, const void* const* x, const void* const* dz,
                             float* const* dw, float* const* part, const ConvShape& s,
                             hipStream_t st, ReduceJob* const* defer);

namespace {


// ---------------------------------------------------------------- 16-byte packs

template <typename T> struct Pk;
template <> struct Pk<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void un(uint4 v, float* f) {
    const uint32_t* d = &v.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[2 * i] = bf2f(d[i] & 0xffffu); f[2 * i + 1] = bf2f(d[i] >> 16); }
  }
  static __device__ __forceinline__ uint4 pk(const float* f) {
    uint4 v;
    uint32_t* d = &v.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = f2bf(f[2 * i]) | (f2bf(f[2 * i + 1]) << 16);
    return v;
  }
};
template <> struct Pk<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void un(uint4 v, float* f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  static __device__ __forceinline__ uint4 pk(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
  }
};

template <typename T> __device__ __forceinline__ uint4 ld16(const T* p) { return *(const uint4*)p; }
template <typename T> __device__ __forceinline__ void st16(T* p, uint4 v) { *(uint4*)p = v; }

// Up to four tensors of each of a launch's n (1 .. kMaxGroup) micro-batches;
// blockIdx.y (or .z) selects one.  Unused entries repeat the first.
struct Group {
  const void* a[kMaxGroup];
  const void* b[kMaxGroup];
  const void* c[kMaxGroup];
  void* y[kMaxGroup];
};
Group make_group(int n, void* const* y, const void* const* a, const void* const* b = nullptr,
                 const void* const* c = nullptr) {
  Group g{};
  for (int k = 0; k < kMaxGroup; ++k) {
    const int q = k < n ? k : 0;
    g.y[k] = y[q];
    if (a) g.a[k] = a[q];
    if (b) g.b[k] = b[q];
    if (c) g.c[k] = c[q];
  }
  return g;
}

// ---------------------------------------------------------------- few-output 1x1

// 1x1 convolution with at most kSmallCo output channels (the network head):
// one thread per pixel reads its channels in 16-byte packs.
constexpr int kSmallCo = 4;

template <typename T>
__global__ __launch_bounds__(256) void conv1x1_small_fwd_k(Group io, const T* __restrict__ w,
                                                           const float* __restrict__ b, long P,
                                                           int Cin, int Cout, int relu) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ x = (const T*)pickg(io.a, blockIdx.y);
  T* __restrict__ y = (T*)pickg(io.y, blockIdx.y);
  const long p = (long)blockIdx.x * 256 + threadIdx.x;
  if (p >= P) return;
  float acc[kSmallCo];
#pragma unroll
  for (int co = 0; co < kSmallCo; ++co) acc[co] = (co < Cout && b) ? b[co] : 0.f;
  for (int c0 = 0; c0 < Cin; c0 += N) {
    float xv[N];
    Pk<T>::un(ld16(x + p * Cin + c0), xv);
#pragma unroll
    for (int co = 0; co < kSmallCo; ++co) {
      if (co >= Cout) break;
#pragma unroll
      for (int i = 0; i < N; ++i) acc[co] += xv[i] * Elt<T>::ld(w + (long)co * Cin + c0 + i);
    }
  }
#pragma unroll
  for (int co = 0; co < kSmallCo; ++co) {
    if (co >= Cout) break;
    Elt<T>::st(y + p * Cout + co, relu ? fmaxf(acc[co], 0.f) : acc[co]);
  }
}

// Its data gradient dx[p][ci] = sum_co dz[p][co] w[co][ci]: a thread keeps one
// channel pack's weights and takes PIX pixels, so that a block writes
// whole rows; bound by that write (64 -> 1 at 192 x 192 x 4: 29 us on the
// float32 matrix unit, 8.6 here).  Four pixels, or one where a launch then has
// fewer than 128 blocks (32 -> 4 at 13 x 13 x 9: 4.9 -> 4.1 us).  blockIdx.y is the
// micro-batch.  Needs 256 % (Cin / pack) == 0.
template <typename T, int PIX>
__global__ __launch_bounds__(256) void dgrad1x1_small_k(Group io, const T* __restrict__ w,
                                                        long P, int Cin, int Cout) {
  constexpr int N = Pk<T>::N;
  const int CP = Cin / N, cp = threadIdx.x % CP, nl = 256 / CP;
  const T* __restrict__ dz = (const T*)pickg(io.a, blockIdx.y);
  T* __restrict__ dx = (T*)pickg(io.y, blockIdx.y);
  float wv[kSmallCo][N];
#pragma unroll
  for (int co = 0; co < kSmallCo; ++co)
#pragma unroll
    for (int i = 0; i < N; ++i)
      wv[co][i] = co < Cout ? Elt<T>::ld(w + (long)co * Cin + cp * N + i) : 0.f;
  const long p0 = (long)blockIdx.x * nl * PIX + threadIdx.x / CP;
  float g[PIX][kSmallCo];
#pragma unroll
  for (int u = 0; u < PIX; ++u)
#pragma unroll
    for (int co = 0; co < kSmallCo; ++co) {   // past the end: the last pixel, unused
      const long p = p0 + (long)u * nl < P ? p0 + (long)u * nl : P - 1;
      g[u][co] = Elt<T>::ld(dz + p * Cout + (co < Cout ? co : 0));
    }
#pragma unroll
  for (int u = 0; u < PIX; ++u) {
    const long p = p0 + (long)u * nl;
    if (p >= P) break;
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
#pragma unroll
    for (int co = 0; co < kSmallCo; ++co) {
      if (co >= Cout) break;
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += g[u][co] * wv[co][i];
    }
    st16(dx + p * Cin + cp * N, Pk<T>::pk(acc));
  }
}

// Its weight gradient dW[co][ci] = sum_p dz[p][co] x[p][ci]: block b covers
// pixels [b*rows, (b+1)*rows); thread t takes channel pack t % CP of pixels
// t / CP, t / CP + 256 / CP, ... in order; row lanes are then added in order
// in LDS and part[b][co][ci] is written.  Needs 256 % CP == 0 (CP = Cin / pack).
template <typename T>
__global__ __launch_bounds__(256) void wgrad1x1_small_k(Group io, long P, int Cin, int Cout,
                                                        long rows) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ x = (const T*)pickg(io.a, blockIdx.y);
  const T* __restrict__ dz = (const T*)pickg(io.b, blockIdx.y);
  float* __restrict__ part = (float*)pickg(io.y, blockIdx.y);
  __shared__ float red[256 * N];
  const int CP = Cin / N;
  const int cp = threadIdx.x % CP, rl = threadIdx.x / CP, nl = 256 / CP;
  const long p0 = (long)blockIdx.x * rows, p1 = p0 + rows < P ? p0 + rows : P;
  float acc[kSmallCo][N];
#pragma unroll
  for (int co = 0; co < kSmallCo; ++co)
#pragma unroll
    for (int i = 0; i < N; ++i) acc[co][i] = 0.f;
  for (long p = p0 + rl; p < p1; p += nl) {
    float xv[N];
    Pk<T>::un(ld16(x + p * Cin + cp * N), xv);
#pragma unroll
    for (int co = 0; co < kSmallCo; ++co) {
      if (co >= Cout) break;
      const float g = Elt<T>::ld(dz + p * Cout + co);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[co][i] += g * xv[i];
    }
  }
  const long E = (long)Cout * Cin;
#pragma unroll
  for (int co = 0; co < kSmallCo; ++co) {   // one output channel at a time through LDS
    if (co >= Cout) break;                  // block-uniform
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) red[threadIdx.x * N + i] = acc[co][i];
    __syncthreads();
    if (rl == 0) {
      float sum[N];
#pragma unroll
      for (int i = 0; i < N; ++i) sum[i] = red[cp * N + i];
      for (int l = 1; l < nl; ++l)
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] += red[(l * CP + cp) * N + i];
#pragma unroll
      for (int i = 0; i < N; ++i) part[(long)blockIdx.x * E + (long)co * Cin + cp * N + i] = sum[i];
    }
  }
}

long direct_wgrad_pps(long P) { return P < 256 ? 256 : (P + 63) / 64; }

// ---------------------------------------------------------------- depthwise

template <typename T>
__global__ __launch_bounds__(256) void dw_fwd(const T* __restrict__ x, const T* __restrict__ w,
                                              const float* __restrict__ b, T* __restrict__ y,
                                              long P, int H, int W, int C, int relu) {
  long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= P * C) return;
  int c = e % C;
  long p = e / C;
  int HW = H * W, rem = p % HW, h = rem / W, wq = rem - h * W;
  float acc = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    int hh = h + t / 3 - 1, ww = wq + t % 3 - 1;
    if ((unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W)
      acc += Elt<T>::ld(w + c * 9 + t) * Elt<T>::ld(x + (p + (long)(t / 3 - 1) * W + (t % 3 - 1)) * C + c);
  }
  if (b) acc += b[c];
  if (relu) acc = fmaxf(acc, 0.f);
  Elt<T>::st(y + e, acc);
}

template <typename T>
__global__ __launch_bounds__(256) void dw_dgrad_k(const T* __restrict__ dz, const T* __restrict__ w,
                                                  T* __restrict__ dx, long P, int H, int W, int C) {
  long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= P * C) return;
  int c = e % C;
  long p = e / C;
  int HW = H * W, rem = p % HW, h = rem / W, wq = rem - h * W;
  float acc = 0.f;
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    int dr = t / 3 - 1, dc = t % 3 - 1;
    int hh = h - dr, ww = wq - dc;
    if ((unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W)
      acc += Elt<T>::ld(w + c * 9 + t) * Elt<T>::ld(dz + (p - (long)dr * W - dc) * C + c);
  }
  Elt<T>::st(dx + e, acc);
}

// Depthwise 3x3 over bf16 NHWC with C % 8 == 0 and C / 8 at most 256; a block
// is a whole number of columns (CP threads each, up to 256).
// Thread q of block (chunk, strip) owns column wc = q / CP and channel pack
// cp = q % CP (CP = C / 8, eight channels per 16-byte pack) and produces the
// output rows [h0, h0 + RS) of that column: the 3 x 3 window of input packs
// slides down the rows, three new packs per output row, so each input pack
// is fetched about (RS + 2) / RS times per column and its horizontal
// neighbours come from the same block's loads.  The nine filter taps of the
// thread's eight channels are one contiguous 144-byte run (w is [C][9]).
// FLIP applies the filter rotated by 180 degrees, which is the data
// gradient (dx = dz correlated with the flipped filter); the sum runs over
// the window in row-major order.
// gridDim.z (1 .. kMaxGroup) micro-batches: blockIdx.z selects x[k] / y[k].
// MASK (data gradient only): the result stored is the ReLU backward of the
// layer below, whose output m[k] masks it (its dz), and the block's column
// sums of the stored values go to part[k] (row blockIdx.y gridDim.x +
// blockIdx.x, C floats): that layer's bias-gradient partials (the threads past
// the last column add zeros).
struct DwIo {
  const bf16_t* x[kMaxGroup];
  bf16_t* y[kMaxGroup];
  const bf16_t* m[kMaxGroup];
  float* part[kMaxGroup];
};
template <int RS, bool FLIP, bool MASK = false>
__global__ __launch_bounds__(256) void dw3_rows_k(DwIo io, const bf16_t* __restrict__ w,
                                                  const float* __restrict__ b, int H, int W, int C,
                                                  int relu) {
  const bf16_t* __restrict__ x = pickg(io.x, blockIdx.z);
  bf16_t* __restrict__ y = pickg(io.y, blockIdx.z);
  const int CP = C >> 3;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int wc = q / CP, cp = q - (q / CP) * CP;
  if (!MASK && wc >= W) return;
  const int strips = (H + RS - 1) / RS;
  const int n = blockIdx.y / strips, h0 = (blockIdx.y - n * strips) * RS;
  float wt[9][8];
  {
    const uint4* wp = (const uint4*)(w + (long)cp * 72);
#pragma unroll
    for (int u = 0; u < 9; ++u) {
      float f[8];
      Pk<bf16_t>::un(wp[u], f);
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int e = u * 8 + v, c = e / 9, t = e - (e / 9) * 9;
        wt[FLIP ? 8 - t : t][c] = f[v];
      }
    }
  }
  float bias[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) bias[i] = b ? b[cp * 8 + i] : 0.f;
  // buffer loads over the sample's image: an offset outside it reads zeros,
  // so the halo needs no branches and the next row's loads stay in flight
  // while this row's products run
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(x + (long)n * H * W * C), (short)0, H * W * C * 2, 0x00020000);
  auto ld = [&](int hh, int ww) __attribute__((always_inline)) {
    const bool ok = (unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W;
    const int off = ok ? ((hh * W + ww) * C + cp * 8) * 2 : (int)0x80000000;
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
  };
  uint4 win[3][3], nxt[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    win[0][s] = ld(h0 - 1, wc + s - 1);
    win[1][s] = ld(h0, wc + s - 1);
    win[2][s] = ld(h0 + 1, wc + s - 1);
  }
  const int h1 = wc < W ? min(h0 + RS, H) : h0;   // (MASK) no rows past the last column
  float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // MASK: this thread's column sums
  for (int h = h0; h < h1; ++h) {
#pragma unroll
    for (int s = 0; s < 3; ++s) nxt[s] = ld(h + 2, wc + s - 1);
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        float f[8];
        Pk<bf16_t>::un(win[r][s], f);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = fmaf(wt[r * 3 + s][i], f[i], acc[i]);
      }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] += bias[i];
      if (relu) acc[i] = fmaxf(acc[i], 0.f);
    }
    const long eo = (long)n * H * W * C + ((long)h * W + wc) * C + cp * 8;
    if constexpr (MASK) {
      float mv[8];
      Pk<bf16_t>::un(ld16(pickg(io.m, blockIdx.z) + eo), mv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = mv[i] > 0.f ? acc[i] : 0.f;
      const uint4 o = Pk<bf16_t>::pk(acc);
      st16(y + eo, o);
      Pk<bf16_t>::un(o, acc);   // the bias gradient sums the stored (rounded) dz
#pragma unroll
      for (int i = 0; i < 8; ++i) bsum[i] += acc[i];
    } else {
      st16(y + eo, Pk<bf16_t>::pk(acc));
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      win[0][s] = win[1][s];
      win[1][s] = win[2][s];
      win[2][s] = nxt[s];
    }
  }
  if constexpr (MASK) {
    // the block's column sums: lanes of one channel pack added in order of
    // their column
    __shared__ float red[256 * 8];
#pragma unroll
    for (int i = 0; i < 8; ++i) red[threadIdx.x * 8 + i] = bsum[i];
    __syncthreads();
    if ((int)threadIdx.x < CP) {
      float s8[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) s8[i] = red[threadIdx.x * 8 + i];
      for (int l = 1; l < (int)blockDim.x / CP; ++l)
#pragma unroll
        for (int i = 0; i < 8; ++i) s8[i] += red[(l * CP + threadIdx.x) * 8 + i];
      float* pr = pickg(io.part, blockIdx.z) + ((long)blockIdx.y * gridDim.x + blockIdx.x) * C +
                  cp * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = s8[i];
    }
  }
}

// Depthwise 3x3 weight-gradient partials over bf16 NHWC (same shape rules
// as dw3_rows_k).  Thread (column, pack) of block (chunk, strip) sums
// dz[p] * x[p + tap] over the rows [h0, h0 + RS) of its column for its
// eight channels and nine taps (x through the sliding window, the next
// row's window and dz loaded while the current row's products run); the
// block then adds its column groups in order in LDS, taps 0-4 and
// then 5-8 through one buffer of a 41-float row per thread (the odd row
// length keeps both the writes and the reads free of bank conflicts), and
// writes part[blk][c * 9 + t], blk = blockIdx.y * chunks + chunk.  A block
// takes the strips blockIdx.y, + gridDim.y, .. one after another.  The partials
// are summed in block order afterwards, so the result is deterministic.
// gridDim.z (1 .. kMaxGroup) micro-batches: blockIdx.z selects (x[k],
// dz[k], part[k]).
struct DwWgIo {
  const bf16_t* x[kMaxGroup];
  const bf16_t* dz[kMaxGroup];
  float* part[kMaxGroup];
};
template <int RS>
__global__ __launch_bounds__(256) void dw3_wgrad_rows_k(DwWgIo io, int nb, int H, int W, int C) {
  const bf16_t* __restrict__ x = pickg(io.x, blockIdx.z);
  const bf16_t* __restrict__ dz = pickg(io.dz, blockIdx.z);
  float* __restrict__ part = pickg(io.part, blockIdx.z);
  constexpr int TH = 5;                      // taps per reduction pass
  constexpr int RW = TH * 8 + 1;             // floats per thread row
  __shared__ float red[256][RW];
  const int CP = C >> 3;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int wc = q / CP, cp = q - (q / CP) * CP;
  const int strips = (H + RS - 1) / RS;
  float acc[9][8];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[t][i] = 0.f;
  for (int strip = blockIdx.y; wc < W && strip < nb * strips; strip += gridDim.y) {
    const int n = strip / strips, h0 = (strip - n * strips) * RS;
    // buffer loads over the sample's image: an offset outside it reads
    // zeros, so the halo needs no branches (a branch per load made the
    // compiler wait for every load in flight, the prefetch included)
    const int img = H * W * C * 2;                              // bytes per sample image
    const long sb = (long)n * H * W * C;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(x + sb), (short)0, img, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(dz + sb), (short)0, img, 0x00020000);
    auto ld = [&](int hh, int ww) __attribute__((always_inline)) {
      const bool ok = (unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W;
      const int off = ok ? ((hh * W + ww) * C + cp * 8) * 2 : (int)0x80000000;
      return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
    };
    auto ldz = [&](int hh) __attribute__((always_inline)) {
      const int off = hh < H ? ((hh * W + wc) * C + cp * 8) * 2 : (int)0x80000000;
      return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rz, off, 0, 0));
    };
    const int h1 = min(h0 + RS, H);
    uint4 win[3][3], nxt[3], dzc = ldz(h0);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      win[0][s] = ld(h0 - 1, wc + s - 1);
      win[1][s] = ld(h0, wc + s - 1);
      win[2][s] = ld(h0 + 1, wc + s - 1);
    }
    for (int h = h0; h < h1; ++h) {
      // next row's loads first: they arrive while this row's products run
#pragma unroll
      for (int s = 0; s < 3; ++s) nxt[s] = ld(h + 2, wc + s - 1);
      const uint4 dzn = ldz(h + 1);
      float d[8];
      Pk<bf16_t>::un(dzc, d);
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          float f[8];
          Pk<bf16_t>::un(win[r][s], f);
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[r * 3 + s][i] = fmaf(d[i], f[i], acc[r * 3 + s][i]);
        }
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        win[0][s] = win[1][s];
        win[1][s] = win[2][s];
        win[2][s] = nxt[s];
      }
      dzc = dzn;
    }
  }
  const int E = C * 9, NG = blockDim.x / CP;
  float* out = part + ((long)blockIdx.y * gridDim.x + blockIdx.x) * E;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int t0 = pass * TH, nt = pass ? 9 - TH : TH;
    if (pass) __syncthreads();                 // the first pass's reads are done
#pragma unroll
    for (int t = 0; t < TH; ++t)
      if (t < nt)
#pragma unroll
        for (int i = 0; i < 8; ++i) red[threadIdx.x][t * 8 + i] = acc[t0 + t][i];
    __syncthreads();
    for (int e = threadIdx.x; e < C * nt; e += blockDim.x) {
      const int c = e / nt, t = e - (e / nt) * nt, pk = c >> 3, i = c & 7;
      float s = 0.f;
      for (int g = 0; g < NG; ++g) s += red[g * CP + pk][t * 8 + i];
      out[c * 9 + t0 + t] = s;
    }
  }
}

// Output rows per thread, forward and data gradient: eight, or two where the
// launch then has fewer than 128 blocks and a thread's chain of rows sets its time
// (64 channels at 29 x 23 x 8: 6.8 -> 4.1 us; 40 at 145 x 145 x 2, 120 blocks, 8.4 ->
// 6.2; the sums are the same).
constexpr int kDwRows = 8, kDwFewRows = 2;
constexpr int kDwWgradRows = 8;  // rows per thread of the weight gradient

// The row-window depthwise kernels apply: bf16, whole 16-byte packs, at most
// 256 of them, 16-byte aligned tensors and weights, and a sample image under
// 2 GiB (their buffer loads take 32-bit offsets).
static bool dw3_rows_shape(int nb, int H, int W, int C) {
  return C > 0 && C % 8 == 0 && C / 8 <= 256 && (long)nb * cdiv(H, kDwRows) <= 65535 &&
         2.0 * H * W * C < 2147483648.0;
}
static bool dw3_rows_ok(int dt, int nb, int H, int W, int C, const void* a, const void* b2,
                        const void* c2) {
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return dt == 0 && dw3_rows_shape(nb, H, W, C) && al(a) && al(b2) && al(c2);
}

// Threads of a block (whole columns of C / 8 packs) and blocks along a row.
static int dw3_threads(int C) { return 256 / (C / 8) * (C / 8); }
static int dw3_chunks(int W, int C) { return (int)cdiv((long)W * (C / 8), dw3_threads(C)); }
static bool dw3_few(int n, int nb, int H, int W, int C) {
  return (long)n * nb * cdiv(H, kDwRows) * dw3_chunks(W, C) < 128;
}
// Blocks of the weight gradient along y: one per strip of a sample.  Where
// the pack count divides no 256-thread block, at most 32 blocks in all (one
// for fewer than 256 pixels; they loop over the strips), so that the partials
// and the layer's bias sums take no more room than the per-element kernel's
// 64 splits; 0 where a row alone has more blocks (that kernel runs).
static int dw3_wgrad_gy(int nb, int H, int W, int C) {
  const long strips = (long)nb * cdiv(H, kDwWgradRows);
  if (256 % (C / 8) == 0) return (int)strips;
  const long cap = ((long)nb * H * W < 256 ? 1 : 32) / dw3_chunks(W, C);
  return (int)(strips < cap ? strips : cap);
}

static int dw3_wgrad_blocks(int nb, int H, int W, int C) {
  return dw3_chunks(W, C) * dw3_wgrad_gy(nb, H, W, C);
}

// ---------------------------------------------------------------- elementwise

template <typename T>
__global__ __launch_bounds__(256) void relu_bwd_k(Group io, int relu, long n, int vec) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ dy = (const T*)pickg(io.a, blockIdx.y);
  const T* __restrict__ ds = (const T*)pickg(io.b, blockIdx.y);
  const T* __restrict__ y = (const T*)pickg(io.c, blockIdx.y);
  T* __restrict__ dz = (T*)pickg(io.y, blockIdx.y);
  long e0 = ((long)blockIdx.x * 256 + threadIdx.x) * N;
  if (e0 >= n) return;
  if (vec && e0 + N <= n) {
    float a[N], s[N], m[N];
    Pk<T>::un(ld16(dy + e0), a);
    if (ds) {
      Pk<T>::un(ld16(ds + e0), s);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] += s[i];
    }
    if (relu) {
      Pk<T>::un(ld16(y + e0), m);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = m[i] > 0.f ? a[i] : 0.f;
    }
    st16(dz + e0, Pk<T>::pk(a));
  } else {
    for (long e = e0; e < n && e < e0 + N; ++e) {
      float a = Elt<T>::ld(dy + e);
      if (ds) a += Elt<T>::ld(ds + e);
      if (relu && !(Elt<T>::ld(y + e) > 0.f)) a = 0.f;
      Elt<T>::st(dz + e, a);
    }
  }
}

// dz = (dy [+ dskip]) * [y > 0] with the bias gradient's column partial sums
// fused in: block b covers rows [b*rows, (b+1)*rows); thread t handles the
// 16-byte channel pack t % CP for rows t / CP, t / CP + nl, ...
// (serial, fixed order); row lanes are then added in order in LDS and
// part[b][c] is written.  A block is CP nl threads, nl = 256 / CP row lanes
// (CP = C / pack, at most 256): all 256 where CP is a power of two.  A launch
// covers gridDim.y (1 .. kMaxGroup) micro-batches of the same shape;
// blockIdx.y selects the pointer set.
template <typename T>
struct RbPtrs {
  const T* dy;   // the incoming gradient (the pool gradient for the pooled kernel)
  const T* ds;
  const T* y;
  T* dz;
  float* part;
};
template <typename T>
struct RbGroup {   // pointer set k of each field is micro-batch k's
  const T* dy[kMaxGroup];
  const T* ds[kMaxGroup];
  const T* y[kMaxGroup];
  T* dz[kMaxGroup];
  float* part[kMaxGroup];
};
// The pointer set of group entry blockIdx.y.
template <typename T>
__device__ __forceinline__ RbPtrs<T> rb_pick(const RbGroup<T>& a) {
  const int k = blockIdx.y;
  return RbPtrs<T>{pickg(a.dy, k), pickg(a.ds, k), pickg(a.y, k), pickg(a.dz, k), pickg(a.part, k)};
}

template <typename T>
__global__ __launch_bounds__(256) void relu_bwd_bias_k(RbGroup<T> ga, int relu, long P, int C,
                                                       long rows) {
  const RbPtrs<T> g = rb_pick(ga);
  const T* __restrict__ dy = g.dy;
  const T* __restrict__ ds = g.ds;
  const T* __restrict__ y = g.y;
  T* __restrict__ dz = g.dz;
  float* __restrict__ part = g.part;
  constexpr int N = Pk<T>::N;
  __shared__ float red[256 * N];
  const int CP = C / N;
  const int cp = threadIdx.x % CP, rl = threadIdx.x / CP, nl = blockDim.x / CP;
  const long p0 = (long)blockIdx.x * rows, p1 = p0 + rows < P ? p0 + rows : P;
  float sum[N];
#pragma unroll
  for (int i = 0; i < N; ++i) sum[i] = 0.f;
  for (long p = p0 + rl; p < p1; p += nl) {
    const long e = p * C + cp * N;
    float a[N], s2[N], m[N];
    Pk<T>::un(ld16(dy + e), a);
    if (ds) {
      Pk<T>::un(ld16(ds + e), s2);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] += s2[i];
    }
    if (relu) {
      Pk<T>::un(ld16(y + e), m);
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = m[i] > 0.f ? a[i] : 0.f;
    }
    uint4 o = Pk<T>::pk(a);
    st16(dz + e, o);
    Pk<T>::un(o, a);   // the bias gradient sums the stored (rounded) dz
#pragma unroll
    for (int i = 0; i < N; ++i) sum[i] += a[i];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) red[threadIdx.x * N + i] = sum[i];
  __syncthreads();
  if (rl == 0) {
    for (int l = 1; l < nl; ++l)
#pragma unroll
      for (int i = 0; i < N; ++i) sum[i] += red[(l * CP + cp) * N + i];
#pragma unroll
    for (int i = 0; i < N; ++i) part[(long)blockIdx.x * C + cp * N + i] = sum[i];
  }
}

// relu_bwd_bias_k for a layer whose output feeds a 2x2/2 max pool: dy is
// the pool gradient dp routed to the first maximal element of each window
// of y.  Block b covers pooled pixels [b*rows, (b+1)*rows); thread t handles
// channel pack t % CP of windows t / CP, t / CP + nl, ... (the four
// pixels of a window in row-major order), then row lanes are added in order
// in LDS and part[b][c] is written.
template <typename T>
__global__ __launch_bounds__(256) void pool_relu_bwd_bias_k(RbGroup<T> ga, int relu, int nb,
                                                            int H, int W, int C, long rows) {
  const RbPtrs<T> gp = rb_pick(ga);
  const T* __restrict__ dp = gp.dy;
  const T* __restrict__ ds = gp.ds;
  const T* __restrict__ y = gp.y;
  T* __restrict__ dz = gp.dz;
  float* __restrict__ part = gp.part;
  constexpr int N = Pk<T>::N;
  __shared__ float red[256 * N];
  const int CP = C / N;
  const int cp = threadIdx.x % CP, rl = threadIdx.x / CP, nl = blockDim.x / CP;
  const int H2 = H / 2, W2 = W / 2;
  const long P2 = (long)nb * H2 * W2;
  const long q0 = (long)blockIdx.x * rows, q1 = q0 + rows < P2 ? q0 + rows : P2;
  float sum[N];
#pragma unroll
  for (int i = 0; i < N; ++i) sum[i] = 0.f;
  for (long q = q0 + rl; q < q1; q += nl) {
    const int w2 = q % W2;
    const long r = q / W2;
    const int h2 = r % H2, n = r / H2;
    const long o = (((long)n * H + 2 * h2) * W + 2 * w2) * C + cp * N;
    const long off[4] = {0, C, (long)W * C, (long)W * C + C};
    float v[4][N], g[N], a[4][N];
#pragma unroll
    for (int k = 0; k < 4; ++k) Pk<T>::un(ld16(y + o + off[k]), v[k]);
    Pk<T>::un(ld16(dp + q * C + cp * N), g);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int arg = 0;
      float best = v[0][i];
#pragma unroll
      for (int k = 1; k < 4; ++k)
        if (v[k][i] > best) { best = v[k][i]; arg = k; }
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k][i] = k == arg ? g[i] : 0.f;
    }
    if (ds) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float s2[N];
        Pk<T>::un(ld16(ds + o + off[k]), s2);
#pragma unroll
        for (int i = 0; i < N; ++i) a[k][i] += s2[i];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (relu) {
#pragma unroll
        for (int i = 0; i < N; ++i) a[k][i] = v[k][i] > 0.f ? a[k][i] : 0.f;
      }
      const uint4 o16 = Pk<T>::pk(a[k]);
      st16(dz + o + off[k], o16);
      Pk<T>::un(o16, a[k]);   // the bias gradient sums the stored (rounded) dz
#pragma unroll
      for (int i = 0; i < N; ++i) sum[i] += a[k][i];
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) red[threadIdx.x * N + i] = sum[i];
  __syncthreads();
  if (rl == 0) {
    for (int l = 1; l < nl; ++l)
#pragma unroll
      for (int i = 0; i < N; ++i) sum[i] += red[(l * CP + cp) * N + i];
#pragma unroll
    for (int i = 0; i < N; ++i) part[(long)blockIdx.x * C + cp * N + i] = sum[i];
  }
}

// Column sums of a P x C matrix: block (cg, pb) sums rows [pb*rows, ...) for
// channels cg*64 .. +63, 256 / (channels) row lanes, combined in fixed order (a
// one-channel head then has 256 lanes at work: 4 of them took 25 us for 147456
// rows, 3.9 now).
template <typename T>
__global__ __launch_bounds__(256) void colsum_k(Group io, long P, int C, long rows) {
  __shared__ float red[256];
  const T* __restrict__ a = (const T*)pickg(io.a, blockIdx.z);
  float* __restrict__ part = (float*)pickg(io.y, blockIdx.z);
  const int c0 = blockIdx.x * 64, nc = C - c0 < 64 ? C - c0 : 64;
  const int nl = 256 / nc, col = threadIdx.x % nc, lane = threadIdx.x / nc;
  const long p0 = (long)blockIdx.y * rows, p1 = p0 + rows < P ? p0 + rows : P;
  float s = 0.f;
  if (lane < nl) {
#pragma unroll 4
    for (long p = p0 + lane; p < p1; p += nl) s += Elt<T>::ld(a + p * C + c0 + col);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  int n = nl;
  while (n > 1) {                                               // block-uniform
    const int h = (n + 1) / 2;
    if (lane < n - h) red[threadIdx.x] += red[threadIdx.x + h * nc];
    __syncthreads();
    n = h;
  }
  if (lane == 0) part[(long)blockIdx.y * C + c0 + col] = red[threadIdx.x];
}

// depthwise wgrad partials: thread (c, tap) of split s
template <typename T>
__global__ __launch_bounds__(256) void dw_wgrad_k(const T* __restrict__ x, const T* __restrict__ dz,
                                                  float* __restrict__ part, long P, int H, int W,
                                                  int C, long pps) {
  long E = (long)C * 9;
  long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= E) return;
  int t = e % 9, c = e / 9;
  int dr = t / 3 - 1, dc = t % 3 - 1;
  long ps = (long)blockIdx.y * pps, pe = ps + pps < P ? ps + pps : P;
  int HW = H * W;
  float acc = 0.f;
  for (long p = ps; p < pe; ++p) {
    int rem = p % HW, h = rem / W, wq = rem - h * W;
    int hh = h + dr, ww = wq + dc;
    if ((unsigned)hh >= (unsigned)H || (unsigned)ww >= (unsigned)W) continue;
    acc += Elt<T>::ld(dz + p * C + c) * Elt<T>::ld(x + (p + (long)dr * W + dc) * C + c);
  }
  part[(long)blockIdx.y * E + e] = acc;
}

// ---------------------------------------------------------------- pool

// The pool and upsample kernels move every byte once and are bound by that; a
// thread takes one channel pack of a 2 x 2 block of pixels, indexed in 32 bits
// (a 64-bit division by each of three sizes took as long as the loads: 64 + 64
// channels at 192 x 192 x 4 upsampled in 13.7 us, 10.9 now).
struct Quad {
  int cp, w2, h2, n;
};
__device__ __forceinline__ Quad quad_of(unsigned e, unsigned CP, unsigned W2, unsigned H2) {
  const unsigned r = e / CP, q = r / W2, n = q / H2;
  return {(int)(e - r * CP), (int)(r - q * W2), (int)(q - n * H2), (int)n};
}

// 2x2/2 max pool of gridDim.y micro-batches.
template <typename T>
__global__ __launch_bounds__(256) void maxpool_fwd_k(Group io, unsigned total, int H, int W, int C) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ x = (const T*)pickg(io.a, blockIdx.y);
  T* __restrict__ y = (T*)pickg(io.y, blockIdx.y);
  const unsigned e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const Quad q = quad_of(e, C / N, W / 2, H / 2);
  const T* base = x + (((long)q.n * H + 2 * q.h2) * W + 2 * q.w2) * C + q.cp * N;
  float m[N], v[N];
  Pk<T>::un(ld16(base), m);
  const long off[3] = {C, (long)W * C, (long)W * C + C};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Pk<T>::un(ld16(base + off[k]), v);
#pragma unroll
    for (int i = 0; i < N; ++i) m[i] = v[i] > m[i] ? v[i] : m[i];
  }
  st16(y + (long)e * N, Pk<T>::pk(m));
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_bwd_k(Group io, unsigned total, int H, int W, int C) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ x = (const T*)pickg(io.a, blockIdx.y);
  const T* __restrict__ dy = (const T*)pickg(io.b, blockIdx.y);
  T* __restrict__ dx = (T*)pickg(io.y, blockIdx.y);
  const unsigned e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const Quad q = quad_of(e, C / N, W / 2, H / 2);
  const long o = (((long)q.n * H + 2 * q.h2) * W + 2 * q.w2) * C + q.cp * N;
  const long off[4] = {0, C, (long)W * C, (long)W * C + C};
  float v[4][N], g[N];
#pragma unroll
  for (int k = 0; k < 4; ++k) Pk<T>::un(ld16(x + o + off[k]), v[k]);
  Pk<T>::un(ld16(dy + (long)e * N), g);
  float out[4][N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    int arg = 0;
    float best = v[0][i];
#pragma unroll
    for (int k = 1; k < 4; ++k)
      if (v[k][i] > best) { best = v[k][i]; arg = k; }
#pragma unroll
    for (int k = 0; k < 4; ++k) out[k][i] = (k == arg) ? g[i] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) st16(dx + o + off[k], Pk<T>::pk(out[k]));
}

// ---------------------------------------------------------------- upsample-concat

// io.a: prev, io.b: skip, io.y: the concatenation.
template <typename T>
__global__ __launch_bounds__(256) void upcat_fwd_k(Group io, unsigned total, int H, int W, int C1,
                                                   int C2) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ prev = (const T*)pickg(io.a, blockIdx.y);
  const T* __restrict__ skip = (const T*)pickg(io.b, blockIdx.y);
  T* __restrict__ out = (T*)pickg(io.y, blockIdx.y);
  const unsigned e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int C = C1 + C2;
  const Quad q = quad_of(e, C / N, W / 2, H / 2);
  const int c = q.cp * N;
  const long p0 = ((long)q.n * H + 2 * q.h2) * W + 2 * q.w2;
  const long off[4] = {0, 1, W, (long)W + 1};
  uint4 v[4];
  if (c < C1) {
    v[0] = ld16(prev + (((long)q.n * (H / 2) + q.h2) * (W / 2) + q.w2) * C1 + c);
    v[1] = v[2] = v[3] = v[0];
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = ld16(skip + (p0 + off[k]) * C2 + (c - C1));
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) st16(out + (p0 + off[k]) * C + c, v[k]);
}

// io.a: dcat, io.y: dprev (sums of the 2 x 2 blocks), io.b: dskip (written).
template <typename T>
__global__ __launch_bounds__(256) void upcat_bwd_k(Group io, unsigned total, int H, int W, int C1,
                                                   int C2) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ dcat = (const T*)pickg(io.a, blockIdx.y);
  T* __restrict__ dprev = (T*)pickg(io.y, blockIdx.y);
  T* __restrict__ dskip = (T*)const_cast<void*>(pickg(io.b, blockIdx.y));
  const unsigned e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int C = C1 + C2;
  const Quad q = quad_of(e, C / N, W / 2, H / 2);
  const int c = q.cp * N;
  const long p0 = ((long)q.n * H + 2 * q.h2) * W + 2 * q.w2;
  const long off[4] = {0, 1, W, (long)W + 1};
  uint4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = ld16(dcat + (p0 + off[k]) * C + c);
  if (c < C1) {
    float sum[N], t[N];
    Pk<T>::un(v[0], sum);
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      Pk<T>::un(v[k], t);
#pragma unroll
      for (int i = 0; i < N; ++i) sum[i] += t[i];
    }
    st16(dprev + (((long)q.n * (H / 2) + q.h2) * (W / 2) + q.w2) * C1 + c, Pk<T>::pk(sum));
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) st16(dskip + (p0 + off[k]) * C2 + (c - C1), v[k]);
  }
}

// ---------------------------------------------------------------- loss / accumulate

// Squared differences of micro-batch blockIdx.y (io.a, io.b) and its loss
// gradient (io.y): block b takes
// the packs of 16 bytes b 256 + t, + gridDim.x 256, .. (one element at a time
// where the tensors are not aligned to packs), adds them per thread in order and
// over the block in a tree.
template <typename T>
__global__ __launch_bounds__(256) void mse_k(Group io, float* __restrict__ part, long n,
                                             float inv_numel, int vec) {
  constexpr int N = Pk<T>::N;
  const T* __restrict__ y = (const T*)pickg(io.a, blockIdx.y);
  const T* __restrict__ t = (const T*)pickg(io.b, blockIdx.y);
  T* __restrict__ dy = (T*)pickg(io.y, blockIdx.y);
  __shared__ float red[256];
  float s = 0.f;
  const long n8 = (n + N - 1) / N;
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; q < n8; q += (long)gridDim.x * 256) {
    const long e0 = q * N;
    if (vec && e0 + N <= n) {
      float a[N], b[N];
      Pk<T>::un(ld16(y + e0), a);
      Pk<T>::un(ld16(t + e0), b);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float d = a[i] - b[i];
        s += d * d;
        a[i] = 2.0f * d * inv_numel;
      }
      st16(dy + e0, Pk<T>::pk(a));
    } else {
      for (long e = e0; e < n && e < e0 + N; ++e) {
        const float d = Elt<T>::ld(y + e) - Elt<T>::ld(t + e);
        s += d * d;
        Elt<T>::st(dy + e, 2.0f * d * inv_numel);
      }
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// *out = scale sum of n partial sums: thread t adds t, t + 256, .. in order,
// the threads meet in a tree.
__global__ __launch_bounds__(256) void loss_sum_k(const float* __restrict__ a, int n, float scale,
                                                  float* __restrict__ out) {
  __shared__ float red[256];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) s += a[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0] * scale;
}

// acc_k = r_k or acc_k + r_k with r_k = sum_{s < S_k} g_k[s n_k + e], every
// entry in one launch.  Tiles blk0[k] .. blk0[k + 1] - 1 serve entry k.  A
// tile of 1024 threads covers C4 float4 columns with LANES = 1024 / C4
// split lanes; lane l sums s = l, l + LANES, .. in ascending order, then the
// lanes are added pairwise in LDS (lane l takes lane l + h for h = LANES / 2,
// .., 1), with (C4, LANES) a function of S only, so the sum is fixed by the
// shape.
__host__ __device__ __forceinline__ int acc_c4(int S) {
  // about four slices per split lane: C4 = 4096 / S rounded down to a power
  // of two, within 1 .. 1024 (a bias gradient's hundreds of block sums then
  // spread over several tiles instead of one long one)
  int c = 1024;
  while (c > 1 && (long)c * S > 4096) c >>= 1;
  return c;
}

// Columns e .. e + 3 of a row of E floats; one by one where the rows' 16-byte
// packs are not aligned (E % 4, tile-uniform).
__device__ __forceinline__ float4 ld_cols(const float* row, long e, long E) {
  if (E % 4 == 0) return *(const float4*)(row + e);
  return make_float4(row[e], e + 1 < E ? row[e + 1] : 0.f, e + 2 < E ? row[e + 2] : 0.f,
                     e + 3 < E ? row[e + 3] : 0.f);
}
__device__ __forceinline__ void st_cols(float* row, long e, long E, float4 v) {
  if (E % 4 == 0) {
    *(float4*)(row + e) = v;
    return;
  }
  row[e] = v.x;
  if (e + 1 < E) row[e + 1] = v.y;
  if (e + 2 < E) row[e + 2] = v.z;
  if (e + 3 < E) row[e + 3] = v.w;
}

// QB micro-batches at a time: their slices are loaded together and their lanes
// meet in one tree, instead of sixteen chains of loads and barriers one after
// the other (256 x 256 weights in 16 slices and a bias of 784 block sums, sixteen
// micro-batches: 70 us one at a time, 58 four at a time, 37 with half the block
// sums; 30 without the bias).
template <int QB>
__global__ __launch_bounds__(1024) void reduce_accumulate_k(AccBatch b, int overwrite,
                                                            int ntiles) {
  // blocks are persistent over tiles (tile = the block of the layout above),
  // so the entry lookup and the block start are paid once per block
  __shared__ float4 red[QB][1024];
  const int ng = b.ng;
  int k = 0;   // entry of the current tile (tiles only increase)
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    while (k + 1 < b.count && tile >= b.blk0[k + 1]) ++k;
    const long bx = (long)tile - b.blk0[k];
    const long E = b.n[k];
    const int S = b.S[k];
    float* __restrict__ acc = b.acc[k];
    const int C4 = acc_c4(S), LANES = 1024 / C4;
    const int col = threadIdx.x % C4, lane = threadIdx.x / C4;
    const long e4 = (bx * C4 + col) * 4;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 cur = zero;   // the running sum (lane 0)
    for (int q0 = 0; q0 < ng; q0 += QB) {
      float4 r[QB];
#pragma unroll
      for (int q = 0; q < QB; ++q) r[q] = zero;
      if (e4 < E) {
        // four slices of each in flight per step; those past S add zeros
        for (int s = lane; s < S; s += 4 * LANES) {
          float4 t[QB][4];
#pragma unroll
          for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u)
              t[q][u] = s + u * LANES < S && q0 + q < ng
                            ? ld_cols(b.g[k] + (q0 + q) * b.gstride[k] + (long)(s + u * LANES) * E, e4, E)
                            : zero;
#pragma unroll
          for (int q = 0; q < QB; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              r[q].x += t[q][u].x; r[q].y += t[q][u].y; r[q].z += t[q][u].z; r[q].w += t[q][u].w;
            }
        }
      }
      if (LANES > 1) {   // tile-uniform
#pragma unroll
        for (int q = 0; q < QB; ++q) red[q][lane * C4 + col] = r[q];
        __syncthreads();
        for (int h = LANES >> 1; h > 0; h >>= 1) {
          if (lane < h) {
#pragma unroll
            for (int q = 0; q < QB; ++q) {
              const float4 t = red[q][(lane + h) * C4 + col];
              r[q].x += t.x; r[q].y += t.y; r[q].z += t.z; r[q].w += t.w;
              red[q][lane * C4 + col] = r[q];
            }
          }
          __syncthreads();   // (the last one also frees red for the next round)
        }
      }
      if (lane == 0 && e4 < E) {
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          if (q0 + q >= ng) break;
          if (q0 + q > 0) {
            cur.x = cur.x + r[q].x; cur.y = cur.y + r[q].y; cur.z = cur.z + r[q].z; cur.w = cur.w + r[q].w;
          } else if (overwrite) {
            cur = r[q];
          } else {
            const float4 o = ld_cols(acc, e4, E);
            cur.x = o.x + r[q].x; cur.y = o.y + r[q].y; cur.z = o.z + r[q].z; cur.w = o.w + r[q].w;
          }
        }
      }
    }
    if (lane == 0 && e4 < E) st_cols(acc, e4, E, cur);
  }
}

inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// ---------------------------------------------------------------- dispatch

int direct_wgrad_splits(long P) { return (int)((P + direct_wgrad_pps(P) - 1) / direct_wgrad_pps(P)); }

static long relu_bias_rows(long P, int C, int N, int cap);

// The 1x1 path for few output channels (the network head).
static bool small1x1_ok(int dt, const ConvShape& s, const void* x) {
  const int N = dt == 0 ? 8 : 4;
  if (s.taps != 1 || s.cout > kSmallCo || s.cin % N || !al16(x)) return false;
  const int CP = s.cin / N;
  return CP <= 256 && 256 % CP == 0;
}

template <typename T>
static hipError_t launch_dgrad_small(int n, const void* const* dz, const void* w, void* const* dx,
                                     const ConvShape& s, hipStream_t st) {
  const Group io = make_group(n, dx, dz);
  const long P = s.pixels(), nl = 256 / (s.cin / Pk<T>::N);
  if (P == 0) return hipSuccess;
  ProfScope ps("dgrad1x1_small", 2.0 * n * P * s.cout * s.cin,
               (double)sizeof(T) * n * P * (s.cin + s.cout), st);
  if (n * cdiv(P, 4 * nl) < 128)
    TGP_LAUNCH(ps, (dgrad1x1_small_k<T, 1>), dim3(cdiv(P, nl), n), dim3(256), 0, st, io,
               (const T*)w, P, s.cin, s.cout);
  else
    TGP_LAUNCH(ps, (dgrad1x1_small_k<T, 4>), dim3(cdiv(P, 4 * nl), n), dim3(256), 0, st, io,
               (const T*)w, P, s.cin, s.cout);
  return launch_status();
}
static hipError_t conv1x1_small(int dt, int n, const void* const* x, const void* w, const float* b,
                                void* const* y, const ConvShape& s, int relu, hipStream_t st) {
  const long P = s.pixels();
  const Group io = make_group(n, y, x);
  ProfScope ps("conv1x1_small_fwd", 2.0 * n * P * s.cout * s.cin,
               (dt == 0 ? 2.0 : 4.0) * n * P * (s.cin + s.cout), st);
  if (dt == 0)
    TGP_LAUNCH(ps, conv1x1_small_fwd_k<bf16_t>, dim3(cdiv(P, 256), n), dim3(256), 0, st, io,
               (const bf16_t*)w, b, P, s.cin, s.cout, relu);
  else
    TGP_LAUNCH(ps, conv1x1_small_fwd_k<float>, dim3(cdiv(P, 256), n), dim3(256), 0, st, io,
               (const float*)w, b, P, s.cin, s.cout, relu);
  return launch_status();
}

// The weight gradient's sums of n micro-batches, left pending in defer[k].
static hipError_t wgrad1x1_small(int dt, int n, const void* const* x, const void* const* dz,
                                 float* const* dw, float* const* part, const ConvShape& s,
                                 hipStream_t st, ReduceJob* const* defer) {
  const long P = s.pixels(), E = (long)s.cout * s.cin;
  const long rows = relu_bias_rows(P, s.cin, dt == 0 ? 8 : 4, 1024);
  const int nbk = cdiv(P, rows);
  const Group io = make_group(n, (void* const*)part, x, dz);
  {
    ProfScope ps("wgrad1x1_small", 2.0 * n * P * E,
                 n * ((dt == 0 ? 2.0 : 4.0) * P * (s.cin + s.cout) + 4.0 * nbk * E), st);
    if (dt == 0)
      TGP_LAUNCH(ps, wgrad1x1_small_k<bf16_t>, dim3(nbk, n), dim3(256), 0, st, io, P, s.cin, s.cout,
                 rows);
    else
      TGP_LAUNCH(ps, wgrad1x1_small_k<float>, dim3(nbk, n), dim3(256), 0, st, io, P, s.cin, s.cout,
                 rows);
  }
  const hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{part[k], dw[k], E, nbk};
  return hipSuccess;
}

static hipError_t dgrad1x1_small(int dt, int n, const void* const* dz, const void* w,
                                 void* const* dx, const ConvShape& s, hipStream_t st) {
  return dt == 0 ? launch_dgrad_small<bf16_t>(n, dz, w, dx, s, st)
                 : launch_dgrad_small<float>(n, dz, w, dx, s, st);
}

hipError_t conv_forward(int dt, const void* x, const void* w, const float* b, void* y,
                        const ConvShape& s, int relu, float* part, size_t part_cap,
                        hipStream_t st) {
  if (mfma_fwd_ok(dt, s))
    return conv_forward_mfma(x, w, b, y, s, relu, part, part_cap, st);
  if (small1x1_ok(dt, s, x)) return conv1x1_small(dt, 1, &x, w, b, &y, s, relu, st);
  if (conv_stem_ok(dt, s)) return conv_stem_forward(1, &x, w, b, &y, s, relu, st);
  return conv_gen_forward(dt, 1, &x, w, b, &y, s, relu, false, st);
}

bool conv_dgrad_uses_wt(int dt, const ConvShape& s, int n_max) {
  const ConvShape t{s.nb, s.H, s.W, s.cout, s.cin, s.taps};
  return mfma_fwd_ok(dt, t) && !conv_dgrad_tile_now(t, n_max);
}

hipError_t conv_dgrad(int dt, const void* dz, const void* w, const void* wt, void* dx,
                      const ConvShape& s, float* part, size_t part_cap, hipStream_t st) {
  const ConvShape t{s.nb, s.H, s.W, s.cout, s.cin, s.taps};
  if (mfma_fwd_ok(dt, t)) {
    if (!wt || conv_dgrad_tile_now(t, 1))
      return conv_dgrad_tile(1, &dz, w, &dx, t, &part, part_cap, st);
    return conv_forward_mfma(dz, wt, nullptr, dx, t, 0, part, part_cap, st);
  }
  if (small1x1_ok(dt, s, dx)) return dgrad1x1_small(dt, 1, &dz, w, &dx, s, st);
  return conv_gen_forward(dt, 1, &dz, w, nullptr, &dx, t, 0, true, st);
}

size_t conv_wgrad_partial_floats(int dt, const ConvShape& s) {
  if (mfma_wgrad_ok(dt, s)) return wgrad_mfma_partial_floats(s);
  const int N = dt == 0 ? 8 : 4;
  if (small1x1_ok(dt, s, (const void*)16)) {   // (alignment is checked per call)
    const size_t direct = conv_gen_wgrad_partial_floats(s);
    const size_t small = (size_t)cdiv(s.pixels(), relu_bias_rows(s.pixels(), s.cin, N, 1024)) * s.cout * s.cin;
    return direct > small ? direct : small;
  }
  return conv_stem_ok(dt, s) ? conv_stem_wgrad_partial_floats(s) : conv_gen_wgrad_partial_floats(s);
}

hipError_t conv_wgrad(int dt, const void* x, const void* dz, float* dw, float* partial,
                      const ConvShape& s, hipStream_t st, ReduceJob* defer) {
  if (!defer) return hipErrorInvalidValue;
  if (mfma_wgrad_ok(dt, s)) return conv_wgrad_mfma(x, dz, dw, partial, s, st, defer);
  return small1x1_ok(dt, s, x) ? wgrad1x1_small(dt, 1, &x, &dz, &dw, &partial, s, st, &defer)
         : conv_stem_ok(dt, s) ? conv_stem_wgrad_launch(1, &x, &dz, &dw, &partial, s, st, &defer)
                               : conv_gen_wgrad_launch(dt, 1, &x, &dz, &dw, &partial, s, st, &defer);
}

hipError_t conv_forward_n(int dt, int n, const void* const* x, const void* w, const float* b,
                          void* const* y, const ConvShape& s, int relu, float* const* part,
                          size_t part_cap, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  if (mfma_fwd_ok(dt, s))
    return conv_forward_mfma_n(n, x, w, b, y, s, relu, part, part_cap, st);
  if (conv_stem_ok(dt, s)) return conv_stem_forward(n, x, w, b, y, s, relu, st);
  bool small = false;
  for (int k = 0; k < n; ++k) small = small || small1x1_ok(dt, s, x[k]);
  if (!small) return conv_gen_forward(dt, n, x, w, b, y, s, relu, false, st);
  bool all = true;
  for (int k = 0; k < n; ++k) all = all && small1x1_ok(dt, s, x[k]);
  if (all) return conv1x1_small(dt, n, x, w, b, y, s, relu, st);
  for (int k = 0; k < n; ++k) {
    const hipError_t e = conv_forward(dt, x[k], w, b, y[k], s, relu, part[k], part_cap, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t conv_dgrad_n(int dt, int n, const void* const* dz, const void* w, const void* wt,
                        void* const* dx, const ConvShape& s, float* const* part,
                        size_t part_cap, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const ConvShape t{s.nb, s.H, s.W, s.cout, s.cin, s.taps};
  if (mfma_fwd_ok(dt, t)) {
    if (!wt || conv_dgrad_tile_now(t, n))
      return conv_dgrad_tile(n, dz, w, dx, t, part, part_cap, st);
    return conv_forward_mfma_n(n, dz, wt, nullptr, dx, t, 0, part, part_cap, st);
  }
  bool small = true;
  for (int k = 0; k < n; ++k) small = small && small1x1_ok(dt, s, dx[k]);
  if (small) return dgrad1x1_small(dt, n, dz, w, dx, s, st);
  return conv_gen_forward(dt, n, dz, w, nullptr, dx, t, 0, true, st);
}

hipError_t conv_wgrad_n(int dt, int n, const void* const* x, const void* const* dz,
                        float* const* dw, float* const* part, const ConvShape& s, hipStream_t st,
                        ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  for (int k = 0; k < n; ++k)
    if (!defer[k]) return hipErrorInvalidValue;
  if (mfma_wgrad_ok(dt, s)) return conv_wgrad_mfma_n(n, x, dz, dw, part, s, st, defer);
  if (conv_stem_ok(dt, s)) return conv_stem_wgrad_launch(n, x, dz, dw, part, s, st, defer);
  bool small = false;
  for (int k = 0; k < n; ++k) small = small || small1x1_ok(dt, s, x[k]);
  if (!small) return conv_gen_wgrad_launch(dt, n, x, dz, dw, part, s, st, defer);
  bool all = true;
  for (int k = 0; k < n; ++k) all = all && small1x1_ok(dt, s, x[k]);
  if (all) return wgrad1x1_small(dt, n, x, dz, dw, part, s, st, defer);
  for (int k = 0; k < n; ++k) {
    const hipError_t e = conv_wgrad(dt, x[k], dz[k], dw[k], part[k], s, st, defer[k]);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool dw_rows_ok(int dt, int nb, int H, int W, int C, const void* a, const void* b,
                const void* c) {
  return dw3_rows_ok(dt, nb, H, W, C, a, b, c);
}

bool dw_wgrad_rows_ok(int dt, int nb, int H, int W, int C, const void* a, const void* b,
                      const void* c) {
  return dw3_rows_ok(dt, nb, H, W, C, a, b, c) && dw3_wgrad_gy(nb, H, W, C) > 0;
}

hipError_t dw_forward_n(int n, const void* const* x, const void* w, const float* b,
                        void* const* y, int nb, int H, int W, int C, int relu, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const long P = (long)nb * H * W;
  if (P == 0) return hipSuccess;
  DwIo io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.y[k] = (bf16_t*)y[k < n ? k : 0];
  }
  const bool few = dw3_few(n, nb, H, W, C);
  const dim3 g((unsigned)dw3_chunks(W, C), (unsigned)(nb * cdiv(H, few ? kDwFewRows : kDwRows)), n);
  ProfScope ps("dw3_rows_fwd", n * 18.0 * P * C, n * 4.0 * P * C, st);
  if (few)
    TGP_LAUNCH(ps, (dw3_rows_k<kDwFewRows, false>), g, dim3(dw3_threads(C)), 0, st, io,
               (const bf16_t*)w, b, H, W, C, relu);
  else
    TGP_LAUNCH(ps, (dw3_rows_k<kDwRows, false>), g, dim3(dw3_threads(C)), 0, st, io,
               (const bf16_t*)w, b, H, W, C, relu);
  return launch_status();
}

hipError_t dw_dgrad_n(int n, const void* const* dz, const void* w, void* const* dx, int nb,
                      int H, int W, int C, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const long P = (long)nb * H * W;
  if (P == 0) return hipSuccess;
  DwIo io;
  for (int k = 0; k < kMaxGroup; ++k) {
    io.x[k] = (const bf16_t*)dz[k < n ? k : 0];
    io.y[k] = (bf16_t*)dx[k < n ? k : 0];
  }
  const bool few = dw3_few(n, nb, H, W, C);
  const dim3 g((unsigned)dw3_chunks(W, C), (unsigned)(nb * cdiv(H, few ? kDwFewRows : kDwRows)), n);
  ProfScope ps("dw3_rows_dgrad", n * 18.0 * P * C, n * 4.0 * P * C, st);
  if (few)
    TGP_LAUNCH(ps, (dw3_rows_k<kDwFewRows, true>), g, dim3(dw3_threads(C)), 0, st, io,
               (const bf16_t*)w, (const float*)nullptr, H, W, C, 0);
  else
    TGP_LAUNCH(ps, (dw3_rows_k<kDwRows, true>), g, dim3(dw3_threads(C)), 0, st, io,
               (const bf16_t*)w, (const float*)nullptr, H, W, C, 0);
  return launch_status();
}

bool dw_dgrad_mask_ok(int nb, int H, int W, int C) {
  return dw3_rows_shape(nb, H, W, C) && 2.0 * nb * H * W * C < 2147483648.0;
}

int dw_dgrad_mask_rows(int nb, int H, int W, int C) {
  return (int)((long)dw3_chunks(W, C) * nb * cdiv(H, kDwRows));
}

hipError_t dw_dgrad_mask_n(int n, const void* const* dz, const void* w, void* const* dx,
                           const void* const* y, float* const* part, int nb, int H, int W, int C,
                           hipStream_t st) {
  if (n < 1 || n > kMaxGroup || !dw_dgrad_mask_ok(nb, H, W, C)) return hipErrorInvalidValue;
  const long P = (long)nb * H * W;
  if (P == 0) return hipSuccess;
  DwIo io;
  for (int k = 0; k < kMaxGroup; ++k) {
    const int q = k < n ? k : 0;
    io.x[k] = (const bf16_t*)dz[q];
    io.y[k] = (bf16_t*)dx[q];
    io.m[k] = (const bf16_t*)y[q];
    io.part[k] = part[q];
    if (!io.x[k] || !io.y[k] || !io.m[k] || !io.part[k]) return hipErrorInvalidValue;
  }
  const dim3 g((unsigned)dw3_chunks(W, C), (unsigned)(nb * cdiv(H, kDwRows)), n);
  ProfScope ps("dw3_rows_dgrad_mask", n * 18.0 * P * C, n * 6.0 * P * C, st);
  TGP_LAUNCH(ps, (dw3_rows_k<kDwRows, true, true>), g, dim3(dw3_threads(C)), 0, st, io, (const bf16_t*)w,
             (const float*)nullptr, H, W, C, 0);
  return launch_status();
}

hipError_t dw_wgrad_n(int n, const void* const* x, const void* const* dz, float* const* dw,
                      float* const* part, int nb, int H, int W, int C, hipStream_t st,
                      ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const long P = (long)nb * H * W;
  const long E = (long)C * 9;
  if (P == 0) return hipSuccess;
  const int S = dw3_wgrad_blocks(nb, H, W, C);
  DwWgIo io;
  for (int k = 0; k < kMaxGroup; ++k) {
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.dz[k] = (const bf16_t*)dz[k < n ? k : 0];
    io.part[k] = part[k < n ? k : 0];
  }
  const dim3 g((unsigned)dw3_chunks(W, C), (unsigned)dw3_wgrad_gy(nb, H, W, C), n);
  {
    ProfScope ps("dw3_wgrad_rows", n * 18.0 * P * C, n * (4.0 * P * C + 4.0 * S * E), st);
    TGP_LAUNCH(ps, (dw3_wgrad_rows_k<kDwWgradRows>), g, dim3(dw3_threads(C)), 0, st, io, nb, H, W, C);
  }
  hipError_t e = launch_status();
  if (defer) {   // left to the caller's accumulation, in the same order
    for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{part[k], dw[k], E, S};
    return e;
  }
  // the sums, two per reduction launch
  for (int k = 0; k < n && e == hipSuccess; k += 2) {
    if (k + 1 < n) {
      const ReduceJob second{part[k + 1], dw[k + 1], E, S};
      e = splitk_reduce_launch(part[k], dw[k], E, S, st, &second);
    } else {
      e = splitk_reduce_launch(part[k], dw[k], E, S, st);
    }
  }
  return e;
}

hipError_t dw_forward(int dt, const void* x, const void* w, const float* b, void* y, int nb,
                      int H, int W, int C, int relu, hipStream_t st) {
  long P = (long)nb * H * W;
  if (dw3_rows_ok(dt, nb, H, W, C, x, w, y))
    return dw_forward_n(1, &x, w, b, &y, nb, H, W, C, relu, st);
  dim3 g(cdiv(P * C, 256));
  ProfScope ps("dw_forward", 18.0 * P * C, (dt == 0 ? 4.0 : 8.0) * P * C, st);
  if (dt == 0)
    TGP_LAUNCH(ps, dw_fwd<bf16_t>, g, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)w,
                       b, (bf16_t*)y, P, H, W, C, relu);
  else
    TGP_LAUNCH(ps, dw_fwd<float>, g, dim3(256), 0, st, (const float*)x, (const float*)w, b,
                       (float*)y, P, H, W, C, relu);
  return launch_status();
}

hipError_t dw_dgrad(int dt, const void* dz, const void* w, void* dx, int nb, int H, int W,
                    int C, hipStream_t st) {
  long P = (long)nb * H * W;
  if (dw3_rows_ok(dt, nb, H, W, C, dz, w, dx))
    return dw_dgrad_n(1, &dz, w, &dx, nb, H, W, C, st);
  dim3 g(cdiv(P * C, 256));
  ProfScope ps("dw_dgrad", 18.0 * P * C, (dt == 0 ? 4.0 : 8.0) * P * C, st);
  if (dt == 0)
    TGP_LAUNCH(ps, dw_dgrad_k<bf16_t>, g, dim3(256), 0, st, (const bf16_t*)dz,
                       (const bf16_t*)w, (bf16_t*)dx, P, H, W, C);
  else
    TGP_LAUNCH(ps, dw_dgrad_k<float>, g, dim3(256), 0, st, (const float*)dz,
                       (const float*)w, (float*)dx, P, H, W, C);
  return launch_status();
}

size_t dw_wgrad_partial_floats(int nb, int H, int W, int C) {
  long P = (long)nb * H * W;
  const size_t direct = (size_t)direct_wgrad_splits(P) * C * 9;
  const size_t rows = dw3_rows_shape(nb, H, W, C) ? (size_t)dw3_wgrad_blocks(nb, H, W, C) * C * 9 : 0;
  return direct > rows ? direct : rows;
}

hipError_t dw_wgrad(int dt, const void* x, const void* dz, float* dw, float* partial, int nb,
                    int H, int W, int C, hipStream_t st) {
  long P = (long)nb * H * W;
  long E = (long)C * 9;
  if (dw_wgrad_rows_ok(dt, nb, H, W, C, x, dz, partial) && P > 0)
    return dw_wgrad_n(1, &x, &dz, &dw, &partial, nb, H, W, C, st);
  long pps = direct_wgrad_pps(P);
  int S = direct_wgrad_splits(P);
  dim3 g(cdiv(E, 256), S);
  {
  ProfScope ps("dw_wgrad", 18.0 * P * C, (dt == 0 ? 4.0 : 8.0) * P * C + 4.0 * S * E, st);
  if (dt == 0)
    TGP_LAUNCH(ps, dw_wgrad_k<bf16_t>, g, dim3(256), 0, st, (const bf16_t*)x,
                       (const bf16_t*)dz, partial, P, H, W, C, pps);
  else
    TGP_LAUNCH(ps, dw_wgrad_k<float>, g, dim3(256), 0, st, (const float*)x,
                       (const float*)dz, partial, P, H, W, C, pps);
  }
  hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  return splitk_reduce_launch(partial, dw, E, S, st);
}

hipError_t relu_backward_n(int dt, int n, const void* const* dy, const void* const* dskip,
                           const void* const* y, void* const* dz, int relu, long numel,
                           hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const int N = dt == 0 ? 8 : 4;
  int vec = 1, skips = 0;
  for (int k = 0; k < n; ++k) {
    if (!al16(dy[k]) || !al16(dz[k]) || !al16(dskip[k]) || (relu && !al16(y[k]))) vec = 0;
    skips += dskip[k] != nullptr;
  }
  const Group io = make_group(n, dz, dy, dskip, y);
  const dim3 g(cdiv(numel, 256L * N), n);
  ProfScope ps("relu_backward", 0.0, (dt == 0 ? 2.0 : 4.0) * numel * (n * (relu ? 3 : 2) + skips), st);
  if (dt == 0)
    TGP_LAUNCH(ps, relu_bwd_k<bf16_t>, g, dim3(256), 0, st, io, relu, numel, vec);
  else
    TGP_LAUNCH(ps, relu_bwd_k<float>, g, dim3(256), 0, st, io, relu, numel, vec);
  return launch_status();
}

static long colsum_rows(long P) { return P < 1024 ? (P < 1 ? 1 : P) : 1024; }
size_t colsum_partial_floats(long P, int C) {
  return (size_t)cdiv(P, colsum_rows(P)) * C;
}

// Threads of a block over CP channel packs: whole rows of packs.
static int pack_threads(int CP) { return 256 / CP * CP; }
// Rows per block of the fused ReLU-backward / bias kernel: about 512 blocks
// (a multiple of the block's row lanes), so deep layers with few pixels and
// many channels still fill the chip.  Where the pack count divides no
// 256-thread block (192 channels: 24 packs), at most `cap` blocks, which the
// plan sets so that their sums fit the room it already had.
static long relu_bias_rows(long P, int C, int N, int cap) {
  const int CP = C / N, nl = 256 / CP;
  // 512 blocks: with 1024 a pass of one micro-batch is no faster (14.1 and 14.2
  // us at 56 x 56 x 256, four samples x 4), and the accumulation reads twice the
  // block sums, its longest chain; with 256 the pass is slower (17 us for 14 in a U-Net of two micro-batches).
  // 1024 where a thread would have more than ten rows, or (up to two packs) whole
  // rounds of rows leave too few blocks: with the accumulation, 64 channels of 205821
  // pixels 20.5 -> 18.9 us; a micro-batch of 16 of 89304 10.2 -> 8.5 in groups of two
  // (alone, where the sums' longer chain shows, 15 -> 18).
  const bool more = CP <= 2 || P > 512L * 10 * nl;
  const long blocks = 256 % CP ? cap : more ? 1024 : 512;
  long r = (P + blocks - 1) / blocks;
  r = (r + nl - 1) / nl * nl;
  return r < nl ? nl : r;
}
bool relu_bias_fusable(int dt, int C, const void* dy, const void* dskip, const void* y,
                       const void* dz) {
  int N = dt == 0 ? 8 : 4;
  return C % N == 0 && C / N <= 256 && al16(dy) && al16(dz) && (!dskip || al16(dskip)) && al16(y);
}
size_t relu_bias_partial_floats(int dt, long P, int C, int cap) {
  const int N = dt == 0 ? 8 : 4;
  if (C % N || C / N > 256) return 0;   // not fusable
  // blocks over P pixels, or over the P / 4 windows of the pooled variant
  const long b1 = cdiv(P, relu_bias_rows(P, C, N, cap));
  const long b2 = cdiv(P / 4, relu_bias_rows(P / 4, C, N, cap));
  return (size_t)(b1 > b2 ? b1 : b2) * C;
}
bool pool_relu_bias_fusable(int dt, int C, int H, int W, const void* dp, const void* dskip,
                            const void* y, const void* dz) {
  return H % 2 == 0 && W % 2 == 0 && H >= 2 && W >= 2 && relu_bias_fusable(dt, C, dp, dskip, y, dz);
}

template <typename T>
static RbPtrs<T> rb_ptrs(const RbArgs& a) {
  return RbPtrs<T>{(const T*)a.dy, (const T*)a.dskip, (const T*)a.y, (T*)a.dz, a.partial};
}
// The group's pointer sets; unused entries repeat the first.
template <typename T>
static RbGroup<T> rb_group(int n, const RbArgs* a) {
  RbGroup<T> g;
  for (int k = 0; k < kMaxGroup; ++k) {
    const RbPtrs<T> p = rb_ptrs<T>(a[k < n ? k : 0]);
    g.dy[k] = p.dy;
    g.ds[k] = p.ds;
    g.y[k] = p.y;
    g.dz[k] = p.dz;
    g.part[k] = p.part;
  }
  return g;
}
// n within 1 .. kMaxGroup, all with or all without a skip gradient.
static bool rb_group_ok(int n, const RbArgs* a) {
  if (n < 1 || n > kMaxGroup) return false;
  for (int k = 1; k < n; ++k)
    if ((a[k].dskip == nullptr) != (a[0].dskip == nullptr)) return false;
  return true;
}

// The bias sums of n launched micro-batches: left pending (defer), or run now.
static hipError_t rb_finish(int n, const RbArgs* a, long C, int nblk, hipStream_t st) {
  ReduceJob jobs[kMaxGroup];
  int now = 0;
  for (int k = 0; k < n; ++k) {
    const ReduceJob job{a[k].partial, a[k].db, C, nblk};
    if (a[k].defer) *a[k].defer = job;
    else jobs[now++] = job;
  }
  return sum_jobs(now, jobs, st, true);
}

hipError_t relu_backward_bias_n(int dt, int n, const RbArgs* a, int relu, long P, int C, int cap,
                                hipStream_t st) {
  if (!rb_group_ok(n, a)) return hipErrorInvalidValue;
  const int N = dt == 0 ? 8 : 4;
  long rows = relu_bias_rows(P, C, N, cap);
  int nb = cdiv(P, rows);
  {
    ProfScope ps("relu_backward_bias", 0.0,
                 n * ((dt == 0 ? 2.0 : 4.0) * P * C * (3 + (a[0].dskip ? 1 : 0) - (relu ? 0 : 1)) +
                      4.0 * nb * C),
                 st);
    if (dt == 0)
      TGP_LAUNCH(ps, relu_bwd_bias_k<bf16_t>, dim3(nb, n), dim3(pack_threads(C / N)), 0, st,
                 rb_group<bf16_t>(n, a), relu, P, C, rows);
    else
      TGP_LAUNCH(ps, relu_bwd_bias_k<float>, dim3(nb, n), dim3(pack_threads(C / N)), 0, st,
                 rb_group<float>(n, a), relu, P, C, rows);
  }
  hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  return rb_finish(n, a, C, nb, st);
}

hipError_t relu_backward_bias(int dt, const void* dy, const void* dskip, const void* y, void* dz,
                              int relu, float* db, float* partial, long P, int C, int cap,
                              hipStream_t st, ReduceJob* defer) {
  const RbArgs a{dy, dskip, y, dz, db, partial, defer};
  return relu_backward_bias_n(dt, 1, &a, relu, P, C, cap, st);
}

hipError_t pool_relu_backward_bias_n(int dt, int n, const RbArgs* a, int relu, int nb, int H,
                                     int W, int C, int cap, hipStream_t st) {
  if (!rb_group_ok(n, a)) return hipErrorInvalidValue;
  for (int k = 0; k < n; ++k)
    if (!pool_relu_bias_fusable(dt, C, H, W, a[k].dy, a[k].dskip, a[k].y, a[k].dz))
      return hipErrorInvalidValue;
  const long P2 = (long)nb * (H / 2) * (W / 2);
  const int N = dt == 0 ? 8 : 4;
  const long rows = relu_bias_rows(P2, C, N, cap);
  const int nbk = cdiv(P2, rows);
  {
    const double esz = dt == 0 ? 2.0 : 4.0;
    ProfScope ps("pool_relu_backward_bias", 0.0,
                 n * (esz * 4.0 * P2 * C * (2 + (a[0].dskip ? 1 : 0)) + esz * P2 * C +
                      4.0 * nbk * C),
                 st);
    if (dt == 0)
      TGP_LAUNCH(ps, pool_relu_bwd_bias_k<bf16_t>, dim3(nbk, n), dim3(pack_threads(C / N)), 0, st,
                 rb_group<bf16_t>(n, a), relu, nb, H, W, C, rows);
    else
      TGP_LAUNCH(ps, pool_relu_bwd_bias_k<float>, dim3(nbk, n), dim3(pack_threads(C / N)), 0, st,
                 rb_group<float>(n, a), relu, nb, H, W, C, rows);
  }
  hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  return rb_finish(n, a, C, nbk, st);
}

hipError_t pool_relu_backward_bias(int dt, const void* dp, const void* dskip, const void* y,
                                   void* dz, int relu, float* db, float* partial, int nb, int H,
                                   int W, int C, int cap, hipStream_t st, ReduceJob* defer) {
  const RbArgs a{dp, dskip, y, dz, db, partial, defer};
  return pool_relu_backward_bias_n(dt, 1, &a, relu, nb, H, W, C, cap, st);
}

hipError_t bias_grad_n(int dt, int n, const void* const* dz, float* const* db,
                       float* const* partial, long P, int C, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const long rows = colsum_rows(P);
  const int nb = cdiv(P, rows);
  const dim3 g(cdiv(C, 64), nb, n);
  {
    const Group io = make_group(n, (void* const*)partial, dz);
    ProfScope ps("bias_colsum", 0.0, n * ((dt == 0 ? 2.0 : 4.0) * P * C + 4.0 * nb * C), st);
    if (dt == 0)
      TGP_LAUNCH(ps, colsum_k<bf16_t>, g, dim3(256), 0, st, io, P, C, rows);
    else
      TGP_LAUNCH(ps, colsum_k<float>, g, dim3(256), 0, st, io, P, C, rows);
  }
  hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  return splitk_reduce_n(n, partial, db, C, nb, st);
}

// Packs of the 2 x 2 blocks of nb images; 0 where a 32-bit index does not reach
// (tensors past the card's memory).
static unsigned quad_total(int nb, int H, int W, int CP) {
  const long t = (long)nb * (H / 2) * (W / 2) * CP;
  return t < (1L << 32) - 256 ? (unsigned)t : 0u;
}

hipError_t maxpool_forward_n(int dt, int n, const void* const* x, void* const* y, int nb, int H,
                             int W, int C, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  for (int k = 0; k < n; ++k)
    if (!x[k] || !y[k]) return hipErrorInvalidValue;
  const unsigned total = quad_total(nb, H, W, C / (dt == 0 ? 8 : 4));
  if (!total) return hipErrorInvalidValue;
  const dim3 g(cdiv(total, 256L), n);
  const Group io = make_group(n, y, x);
  ProfScope ps("maxpool_forward", 0.0, n * (dt == 0 ? 2.0 : 4.0) * nb * H * W * C * 1.25, st);
  if (dt == 0)
    TGP_LAUNCH(ps, maxpool_fwd_k<bf16_t>, g, dim3(256), 0, st, io, total, H, W, C);
  else
    TGP_LAUNCH(ps, maxpool_fwd_k<float>, g, dim3(256), 0, st, io, total, H, W, C);
  return launch_status();
}

hipError_t maxpool_backward_n(int dt, int n, const void* const* x, const void* const* dy,
                              void* const* dx, int nb, int H, int W, int C, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const unsigned total = quad_total(nb, H, W, C / (dt == 0 ? 8 : 4));
  if (!total) return hipErrorInvalidValue;
  const dim3 g(cdiv(total, 256L), n);
  const Group io = make_group(n, dx, x, dy);
  ProfScope ps("maxpool_backward", 0.0, n * (dt == 0 ? 2.0 : 4.0) * nb * H * W * C * 2.25, st);
  if (dt == 0)
    TGP_LAUNCH(ps, maxpool_bwd_k<bf16_t>, g, dim3(256), 0, st, io, total, H, W, C);
  else
    TGP_LAUNCH(ps, maxpool_bwd_k<float>, g, dim3(256), 0, st, io, total, H, W, C);
  return launch_status();
}

hipError_t upcat_forward_n(int dt, int n, const void* const* prev, const void* const* skip,
                           void* const* out, int nb, int H, int W, int C1, int C2,
                           hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const unsigned total = quad_total(nb, H, W, (C1 + C2) / (dt == 0 ? 8 : 4));
  if (!total) return hipErrorInvalidValue;
  const dim3 g(cdiv(total, 256L), n);
  const Group io = make_group(n, out, prev, skip);
  ProfScope ps("upcat_forward", 0.0, n * (dt == 0 ? 2.0 : 4.0) * nb * H * W * (1.25 * C1 + 2.0 * C2), st);
  if (dt == 0)
    TGP_LAUNCH(ps, upcat_fwd_k<bf16_t>, g, dim3(256), 0, st, io, total, H, W, C1, C2);
  else
    TGP_LAUNCH(ps, upcat_fwd_k<float>, g, dim3(256), 0, st, io, total, H, W, C1, C2);
  return launch_status();
}

hipError_t upcat_backward_n(int dt, int n, const void* const* dcat, void* const* dprev,
                            void* const* dskip, int nb, int H, int W, int C1, int C2,
                            hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const unsigned total = quad_total(nb, H, W, (C1 + C2) / (dt == 0 ? 8 : 4));
  if (!total) return hipErrorInvalidValue;
  const dim3 g(cdiv(total, 256L), n);
  const Group io = make_group(n, dprev, dcat, (const void* const*)dskip);
  ProfScope ps("upcat_backward", 0.0, n * (dt == 0 ? 2.0 : 4.0) * nb * H * W * (1.25 * C1 + 2.0 * C2), st);
  if (dt == 0)
    TGP_LAUNCH(ps, upcat_bwd_k<bf16_t>, g, dim3(256), 0, st, io, total, H, W, C1, C2);
  else
    TGP_LAUNCH(ps, upcat_bwd_k<float>, g, dim3(256), 0, st, io, total, H, W, C1, C2);
  return launch_status();
}

// Blocks of one micro-batch's loss: one per 2048 elements (16384 a block and one
// thread adding the blocks up took 18 us for 32768 elements and 32 us for 147456), up
// to 512, two a CU.  At most 64, 512 and 1024 blocks, us a micro-batch in bf16:
// 802816 elements 16.5, 6.0, 6.1; 9437184 42, 10.8, 9.7; 67108864 380, 73, 69.  Eight
// micro-batches of 9437184 in one launch and the launch that adds up the blocks' sums:
// 87 + 3.9, 83 + 7.0, 80 + 12.4.
int mse_blocks(long n) {
  const long b = cdiv(n, 2048);
  return (int)(b < 512 ? b : 512);
}

hipError_t mse_forward_backward_n(int dt, int n, const void* const* y, const void* const* t,
                                  void* const* dy, float* partial, long numel, float inv_numel,
                                  hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  int vec = 1;
  for (int k = 0; k < n; ++k)
    if (!al16(y[k]) || !al16(t[k]) || !al16(dy[k])) vec = 0;
  const Group io = make_group(n, dy, y, t);
  const dim3 g(mse_blocks(numel), n);
  ProfScope ps("mse", 3.0 * n * numel, n * (dt == 0 ? 6.0 : 12.0) * numel, st);
  if (dt == 0)
    TGP_LAUNCH(ps, mse_k<bf16_t>, g, dim3(256), 0, st, io, partial, numel, inv_numel, vec);
  else
    TGP_LAUNCH(ps, mse_k<float>, g, dim3(256), 0, st, io, partial, numel, inv_numel, vec);
  return launch_status();
}

hipError_t loss_finalize(const float* parts, int n, float inv_numel, float* loss,
                         hipStream_t st) {
  ProfScope ps("loss_sum", (double)n, 4.0 * n, st);
  TGP_LAUNCH(ps, loss_sum_k, dim3(1), dim3(256), 0, st, parts, n, inv_numel, loss);
  return launch_status();
}

hipError_t grad_accumulate_batch(AccBatch b, int overwrite, hipStream_t st, const char* name) {
  if (b.count < 0 || b.count > kMaxAcc || b.ng < 1 || b.ng > kMaxGroup) return hipErrorInvalidValue;
  long blocks = 0;
  double bytes = 0;
  int used = 0;
  for (int k = 0; k < b.count; ++k) {
    if (b.n[k] <= 0 || b.S[k] < 1) continue;
    b.acc[used] = b.acc[k]; b.g[used] = b.g[k]; b.gstride[used] = b.gstride[k];
    b.n[used] = b.n[k]; b.S[used] = b.S[k];
    b.blk0[used] = (int)blocks;
    const int C4 = acc_c4(b.S[k]);
    blocks += cdiv(b.n[k], 4L * C4);
    bytes += 4.0 * b.n[k] * ((double)b.S[k] * b.ng + (overwrite ? 1 : 2));
    ++used;
  }
  b.count = used;
  if (used == 0) return hipSuccess;
  if (blocks >= (1L << 31)) return hipErrorInvalidValue;
  ProfScope ps(name, 0.0, bytes, st);
  const unsigned grid = (unsigned)(blocks < 512 ? blocks : 512);   // two blocks per CU
  if (b.ng == 1)
    TGP_LAUNCH(ps, reduce_accumulate_k<1>, dim3(grid), dim3(1024), 0, st, b, overwrite,
               (int)blocks);
  else
    TGP_LAUNCH(ps, reduce_accumulate_k<4>, dim3(grid), dim3(1024), 0, st, b, overwrite,
               (int)blocks);
  return launch_status();
}

hipError_t sum_jobs(int n, const ReduceJob* jobs, hipStream_t st, bool single) {
  if (n < 0 || n > kMaxGroup) return hipErrorInvalidValue;
  AccBatch b;
  b.count = 0;
  b.ng = 1;
  for (int k = 0; k < n; ++k) {
    if (jobs[k].S < (single ? 1 : 2)) continue;
    b.acc[b.count] = jobs[k].out;
    b.g[b.count] = jobs[k].part;
    b.gstride[b.count] = 0;
    b.n[b.count] = jobs[k].E;
    b.S[b.count++] = jobs[k].S;
  }
  return grad_accumulate_batch(b, 1, st, "reduce_now");
}

}  // namespace tgpk
