// 3x3 and 1x1 convolutions on float32 matrix instructions
// (v_mfma_f32_32x32x2_f32): every float32 layer, and bf16 layers whose channel
// counts the bf16 kernels do not take (an RGB image, a one-channel mask).  Any
// sizes; products and sums are float32 throughout (bf16 operands are widened
// as they are loaded, which is exact).
//
// Forward: Y^T[co][p] = sum_k W[co][k] im2col(X)[p][k], k = (tap, channel)
// flattened, so the weights' rows are contiguous and a K step of 32 may run
// over several taps of a thin layer.  The data gradient is the same with the
// source pixel on the other side of the tap and W read across its rows.
// Weight gradient: dW[co][n] = sum_p dZ[p][co] im2col(X)[p][n], n = (tap,
// channel) flattened, over a range of pixels per block; the ranges' slices are
// summed in order afterwards.
//
// A matrix instruction takes 64 cycles here for two operand values a lane, so
// plain register-staged tiles, double-buffered in LDS, keep the matrix cores
// fed; what is left is latency: small layers have few tiles, so the waves of a
// block split the K step between them where there are too few.  The direct
// kernels this replaces computed one output a thread from scalar loads, at 1
// to 2 TFLOP/s (5 in the data gradient).
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {

__device__ __forceinline__ f32x16_t mfma_f32(float a, float b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Four consecutive elements at p (VEC: aligned to them), as float32; only the
// first n of them are read, the rest are zeros.
template <bool VEC>
__device__ __forceinline__ f32x4_t ld4(const float* p, int n) {
  if constexpr (VEC) {
    return n > 0 ? *(const f32x4_t*)p : f32x4_t{};
  } else {
    f32x4_t v{};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) v[e] = p[e];
    return v;
  }
}
template <bool VEC>
__device__ __forceinline__ f32x4_t ld4(const bf16_t* p, int n) {
  f32x4_t v{};
  if constexpr (VEC) {
    if (n > 0) {
      const uint2 u = *(const uint2*)p;
      v = f32x4_t{bf2f(u.x & 0xffffu), bf2f(u.x >> 16), bf2f(u.y & 0xffffu), bf2f(u.y >> 16)};
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) v[e] = bf2f(p[e]);
  }
  return v;
}
template <bool VEC>
__device__ __forceinline__ void st4(float* p, f32x4_t v, int n) {
  if constexpr (VEC) {
    *(f32x4_t*)p = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) p[e] = v[e];
  }
}
template <bool VEC>
__device__ __forceinline__ void st4(bf16_t* p, f32x4_t v, int n) {
  if constexpr (VEC) {
    uint2 o;
    o.x = f2bf(v[0]) | (f2bf(v[1]) << 16);
    o.y = f2bf(v[2]) | (f2bf(v[3]) << 16);
    *(uint2*)p = o;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) p[e] = (bf16_t)f2bf(v[e]);
  }
}

// The n micro-batches of one launch (P pixels each, the same weights).
template <typename T>
struct GenIo {
  const T* x[kMaxGroup];
  T* y[kMaxGroup];
};

constexpr int GBK = 32;            // K step
constexpr int GLD = GBK + 4;       // floats per LDS row: eight rows on distinct bank groups

// CI sum channels, CO output channels.  WCO x WP x KS = 4 waves: a block's
// tile is 32 WCO output channels x 32 WP pixels, and KS waves share a 32 x 32
// tile, each taking every KS-th 8 of a K step; their sums meet in LDS in wave
// order.  VEC: CI and CO are multiples of 4.
template <typename T, int WCO, int WP, int KS, bool DG, bool VEC>
__global__ __launch_bounds__(256) void conv_gen(GenIo<T> io, const T* __restrict__ Wt,
                                                const float* __restrict__ bias, int P, int H, int W,
                                                int CI, int CO, int taps, int relu, int npt) {
  static_assert(WCO * WP * KS == 4, "4 waves");
  constexpr int BN = 32 * WCO, BM = 32 * WP;
  constexpr int AL = BN / 32, BL = BM / 32;      // 4-element loads per thread and K step
  __shared__ __attribute__((aligned(16))) float smem[2][(BN + BM) * GLD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ks = wave % KS, wp = wave / KS % WP, wco = wave / (KS * WP);
  const int nct = (CO + BN - 1) / BN;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int gi = lb / (npt * nct);               // micro-batch (uniform)
  const int t0 = lb - gi * npt * nct;
  const int p0 = (t0 / nct) * BM, co0 = (t0 % nct) * BN;
  const T* __restrict__ X = pickg(io.x, gi);
  T* __restrict__ Y = pickg(io.y, gi);
  const int K = taps * CI;
  const int HW = H * W;

  // B loads: 4 k's (chunk q of the K step) of pixel rows tid / 8 + 32 u
  const int q = tid & 7;
  int ph[BL], pw[BL];
  bool pok[BL];
#pragma unroll
  for (int u = 0; u < BL; ++u) {
    const int p = p0 + (tid >> 3) + 32 * u;
    pok[u] = p < P;
    const int rem = (pok[u] ? p : 0) % HW;
    ph[u] = rem / W;
    pw[u] = rem - ph[u] * W;
  }
  const long xrow = p0 + (tid >> 3);
  f32x4_t ra[AL], rb[BL];
  auto gload = [&](int k0) __attribute__((always_inline)) {
    const int kb = k0 + 4 * q;
    // im2col rows
    if constexpr (VEC) {
      const int tap = kb / CI, c = kb - tap * CI;
      const int dr = taps == 9 ? (DG ? 1 - tap / 3 : tap / 3 - 1) : 0;
      const int dc = taps == 9 ? (DG ? 1 - tap % 3 : tap % 3 - 1) : 0;
#pragma unroll
      for (int u = 0; u < BL; ++u) {
        const bool ok = kb < K && pok[u] && (unsigned)(ph[u] + dr) < (unsigned)H &&
                        (unsigned)(pw[u] + dc) < (unsigned)W;
        rb[u] = ld4<true>(X + (xrow + 32 * u + (long)dr * W + dc) * CI + c, ok ? 4 : 0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < BL; ++u) rb[u] = f32x4_t{};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = kb + e;
        if (k >= K) continue;
        const int tap = k / CI, c = k - tap * CI;
        const int dr = taps == 9 ? (DG ? 1 - tap / 3 : tap / 3 - 1) : 0;
        const int dc = taps == 9 ? (DG ? 1 - tap % 3 : tap % 3 - 1) : 0;
#pragma unroll
        for (int u = 0; u < BL; ++u)
          if (pok[u] && (unsigned)(ph[u] + dr) < (unsigned)H && (unsigned)(pw[u] + dc) < (unsigned)W)
            rb[u][e] = Elt<T>::ld(X + (xrow + 32 * u + (long)dr * W + dc) * CI + c);
      }
    }
    // weights: forward, 4 k's of rows tid / 8 + 32 u; data gradient, 4 output
    // channels of k's k0 + tid / (BN / 4) + (1024 / BN) u
    if constexpr (!DG) {
#pragma unroll
      for (int u = 0; u < AL; ++u) {
        const int co = co0 + (tid >> 3) + 32 * u;
        ra[u] = ld4<VEC>(Wt + (long)co * K + kb, co < CO ? K - kb : 0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < AL; ++u) {
        const int k = k0 + tid / (BN / 4) + (1024 / BN) * u;
        const int tap = k / CI, r = k - tap * CI;               // the layer's output channel r
        const int c = co0 + 4 * (tid % (BN / 4));
        ra[u] = ld4<VEC>(Wt + ((long)r * taps + tap) * CO + c, k < K ? CO - c : 0);
      }
    }
  };
  auto lstore = [&](int buf) __attribute__((always_inline)) {
    float* As = smem[buf];
    float* Bs = smem[buf] + BN * GLD;
    if constexpr (!DG) {
#pragma unroll
      for (int u = 0; u < AL; ++u) *(f32x4_t*)(As + ((tid >> 3) + 32 * u) * GLD + 4 * q) = ra[u];
    } else {
#pragma unroll
      for (int u = 0; u < AL; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          As[(4 * (tid % (BN / 4)) + e) * GLD + tid / (BN / 4) + (1024 / BN) * u] = ra[u][e];
    }
#pragma unroll
    for (int u = 0; u < BL; ++u) *(f32x4_t*)(Bs + ((tid >> 3) + 32 * u) * GLD + 4 * q) = rb[u];
  };

  f32x16_t acc = f32x16_t{};
  gload(0);
  lstore(0);
  __syncthreads();
  const int nk = (K + GBK - 1) / GBK;
  const int h = lane >> 5;
  for (int s = 0; s < nk; ++s) {
    if (s + 1 < nk) gload((s + 1) * GBK);
    const float* As = smem[s & 1] + (wco * 32 + (lane & 31)) * GLD + 4 * h;
    const float* Bs = smem[s & 1] + BN * GLD + (wp * 32 + (lane & 31)) * GLD + 4 * h;
    const int left = K - s * GBK;                // (uniform) k's past K are zeros: left out
#pragma unroll
    for (int j = 0; j < 4; j += KS) {
      const int jj = j + ks;
      if (8 * jj < left) {
        const f32x4_t a = *(const f32x4_t*)(As + 8 * jj);
        const f32x4_t b = *(const f32x4_t*)(Bs + 8 * jj);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma_f32(a[e], b[e], acc);
      }
    }
    if (s + 1 < nk) lstore((s + 1) & 1);
    __syncthreads();
  }
  if constexpr (KS > 1) {
    // each wave's 16 sums per lane; the first of the KS waves adds them up
    float* red = &smem[0][0];
    static_assert(4 * 64 * 17 <= 2 * (BN + BM) * GLD, "sums fit the tiles");
    if (ks) {
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(wave * 64 + lane) * 17 + v] = acc[v];
    }
    __syncthreads();
    if (ks) return;
#pragma unroll
    for (int o = 1; o < KS; ++o)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] += red[((wave + o) * 64 + lane) * 17 + v];
  }
  // element v of lane l: output channel 8 (v / 4) + 4 (l / 32) + v % 4, pixel l % 32
  const int p = p0 + wp * 32 + (lane & 31);
  if (p >= P) return;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int co = co0 + wco * 32 + 8 * g + 4 * h;
    const int n = CO - co;
    if (n <= 0) continue;
    f32x4_t v = f32x4_t{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (bias && e < n) v[e] += bias[co + e];
      if (relu) v[e] = fmaxf(v[e], 0.0f);
    }
    st4<VEC>(Y + (long)p * CO + co, v, n);
  }
}

template <typename T>
struct GenWgIo {
  const T* x[kMaxGroup];
  const T* dz[kMaxGroup];
  float* part[kMaxGroup];
};

// WM x WN = 4 waves: a block's tile is 32 WM output channels x 32 WN columns n
// = (tap, channel), summed over the pixels [split pps, + pps); blocks are
// (micro-batch, split, tile), tile fastest.  VEC: CI and CO multiples of 4.
template <typename T, int WM, int WN, bool VEC>
__global__ __launch_bounds__(256) void conv_gen_wgrad(GenWgIo<T> io, int P, int H, int W, int CI,
                                                      int CO, int taps, int S, int pps) {
  static_assert(WM * WN == 4, "4 waves");
  constexpr int BMc = 32 * WM, BNc = 32 * WN;
  constexpr int LA = BMc + 4, LB = BNc + 4;      // floats per LDS row (a pixel)
  constexpr int AU = BMc / 32, BU = BNc / 32;    // 4-element loads per thread and K step
  constexpr int AC = BMc / 4, BC = BNc / 4;      // chunks per pixel
  __shared__ __attribute__((aligned(16))) float smem[2][GBK * (LA + LB)];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave % WN, wm = wave / WN;
  const int N = taps * CI;
  const int nct = (CO + BMc - 1) / BMc, nnt = (N + BNc - 1) / BNc;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = lb % (nct * nnt), sg = lb / (nct * nnt);
  const int split = sg % S, gi = sg / S;
  const int co0 = (tile / nnt) * BMc, n0 = (tile % nnt) * BNc;
  const T* __restrict__ X = pickg(io.x, gi);
  const T* __restrict__ dZ = pickg(io.dz, gi);
  float* __restrict__ out = pickg(io.part, gi) + (long)split * CO * N;
  const int ps = split * pps, pe = min(P, ps + pps);

  // A: chunk ca of pixels pa + (256 / AC) u; B: chunk cb of pixels pb + (256 / BC) u
  const int ca = tid % AC, pa = tid / AC, cb = tid % BC, pb = tid / BC;
  // column n's tap and channel (VEC: the four columns of a chunk share a tap)
  int dr[4], dc[4], ch[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int n = min(n0 + 4 * cb + e, N - 1);
    const int tap = n / CI;
    ch[e] = n - tap * CI;
    dr[e] = taps == 9 ? tap / 3 - 1 : 0;
    dc[e] = taps == 9 ? tap % 3 - 1 : 0;
  }
  const int nn = N - (n0 + 4 * cb);              // columns left at this chunk
  int bh[BU], bw[BU];                            // coordinates of the B pixels
#pragma unroll
  for (int u = 0; u < BU; ++u) {
    const int rem = (ps + pb + (256 / BC) * u) % (H * W);
    bh[u] = rem / W;
    bw[u] = rem - bh[u] * W;
  }
  f32x4_t ra[AU], rb[BU];
  auto gload = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < AU; ++u) {
      const int p = k0 + pa + (256 / AC) * u, co = co0 + 4 * ca;
      ra[u] = ld4<VEC>(dZ + (long)p * CO + co, p < pe ? CO - co : 0);
    }
#pragma unroll
    for (int u = 0; u < BU; ++u) {
      const int p = k0 + pb + (256 / BC) * u;
      if constexpr (VEC) {
        const bool ok = p < pe && nn > 0 && (unsigned)(bh[u] + dr[0]) < (unsigned)H &&
                        (unsigned)(bw[u] + dc[0]) < (unsigned)W;
        rb[u] = ld4<true>(X + (p + (long)dr[0] * W + dc[0]) * CI + ch[0], ok ? 4 : 0);
      } else {
        rb[u] = f32x4_t{};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (p < pe && e < nn && (unsigned)(bh[u] + dr[e]) < (unsigned)H &&
              (unsigned)(bw[u] + dc[e]) < (unsigned)W)
            rb[u][e] = Elt<T>::ld(X + (p + (long)dr[e] * W + dc[e]) * CI + ch[e]);
      }
      bw[u] += GBK;
      while (bw[u] >= W) {
        bw[u] -= W;
        if (++bh[u] == H) bh[u] = 0;
      }
    }
  };
  auto lstore = [&](int buf) __attribute__((always_inline)) {
    float* As = smem[buf];
    float* Bs = smem[buf] + GBK * LA;
#pragma unroll
    for (int u = 0; u < AU; ++u) *(f32x4_t*)(As + (pa + (256 / AC) * u) * LA + 4 * ca) = ra[u];
#pragma unroll
    for (int u = 0; u < BU; ++u) *(f32x4_t*)(Bs + (pb + (256 / BC) * u) * LB + 4 * cb) = rb[u];
  };

  f32x16_t acc = f32x16_t{};
  const int nk = (pe - ps + GBK - 1) / GBK;
  if (nk > 0) {
    gload(ps);
    lstore(0);
  }
  __syncthreads();
  const int h = lane >> 5;
  for (int s = 0; s < nk; ++s) {
    if (s + 1 < nk) gload(ps + (s + 1) * GBK);
    const float* As = smem[s & 1] + h * LA + wm * 32 + (lane & 31);
    const float* Bs = smem[s & 1] + GBK * LA + h * LB + wn * 32 + (lane & 31);
#pragma unroll
    for (int k = 0; k < GBK / 2; ++k) acc = mfma_f32(As[2 * k * LA], Bs[2 * k * LB], acc);
    if (s + 1 < nk) lstore((s + 1) & 1);
    __syncthreads();
  }
  // element v of lane l: output channel 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
  const int n = n0 + wn * 32 + (lane & 31);
  if (n >= N) return;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int co = co0 + wm * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
    if (co < CO) out[(long)co * N + n] = acc[v];
  }
}

// Tile of a shape: 64 x 64 where four samples give 256 tiles, else 64 x 32 and
// 32 x 32 with the K step split over two and four waves (a few thousand pixels
// of a thin layer are otherwise a few dozen blocks); 32 channels at a time
// where there are no more.  A function of the per-sample shape, so that every
// sample's sums keep their order whatever the micro-batch.
int gen_tile(const ConvShape& s) {
  const long P = 4L * s.H * s.W;
  if (s.cout <= 32) return P / 128 >= 256 ? 3 : 2;
  const long t64 = (P + 63) / 64 * ((s.cout + 63) / 64);
  return t64 >= 256 ? 0 : t64 >= 128 ? 1 : 2;
}

template <typename T, int WCO, int WP, int KS, bool DG, bool VEC>
hipError_t launch_gen_t(const char* name, const GenIo<T>& io, int n, const T* w, const float* b,
                        const ConvShape& s, int relu, hipStream_t st) {
  const long P = s.pixels();
  const int npt = cdiv(P, 32L * WP);
  const long blocks = (long)n * npt * ((s.cout + 32 * WCO - 1) / (32 * WCO));
  if (blocks >= (1L << 31)) return hipErrorInvalidValue;
  ProfScope ps(name, 2.0 * n * P * s.cout * s.taps * s.cin,
               (double)sizeof(T) * (n * P * (s.cin + s.cout) + (double)s.cout * s.taps * s.cin), st);
  TGP_LAUNCH(ps, (conv_gen<T, WCO, WP, KS, DG, VEC>), dim3((unsigned)blocks), dim3(256), 0, st, io,
             w, b, (int)P, s.H, s.W, s.cin, s.cout, s.taps, relu, npt);
  return launch_status();
}
template <typename T, bool DG, bool VEC>
hipError_t launch_gen(int n, const void* const* x, const void* w, const float* b, void* const* y,
                      const ConvShape& s, int relu, hipStream_t st) {
  GenIo<T> io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.x[k] = (const T*)x[k < n ? k : 0];
    io.y[k] = (T*)y[k < n ? k : 0];
  }
  const T* W = (const T*)w;
  switch (gen_tile(s)) {
    case 0: return launch_gen_t<T, 2, 2, 1, DG, VEC>(DG ? "conv_gen_dg<2,2,1>" : "conv_gen<2,2,1>", io, n, W, b, s, relu, st);
    case 1: return launch_gen_t<T, 2, 1, 2, DG, VEC>(DG ? "conv_gen_dg<2,1,2>" : "conv_gen<2,1,2>", io, n, W, b, s, relu, st);
    case 3: return launch_gen_t<T, 1, 4, 1, DG, VEC>(DG ? "conv_gen_dg<1,4,1>" : "conv_gen<1,4,1>", io, n, W, b, s, relu, st);
    default: return launch_gen_t<T, 1, 1, 4, DG, VEC>(DG ? "conv_gen_dg<1,1,4>" : "conv_gen<1,1,4>", io, n, W, b, s, relu, st);
  }
}

}  // namespace

hipError_t conv_gen_forward(int dt, int n, const void* const* x, const void* w, const float* b,
                            void* const* y, const ConvShape& s, int relu, bool dg,
                            hipStream_t st) {
  if (n < 1 || n > kMaxGroup || s.pixels() <= 0) return hipErrorInvalidValue;
  const bool vec = s.cin % 4 == 0 && s.cout % 4 == 0;
#define GEN_GO(T, D, V) launch_gen<T, D, V>(n, x, w, b, y, s, relu, st)
  if (dt == 0)
    return dg ? (vec ? GEN_GO(bf16_t, true, true) : GEN_GO(bf16_t, true, false))
              : (vec ? GEN_GO(bf16_t, false, true) : GEN_GO(bf16_t, false, false));
  return dg ? (vec ? GEN_GO(float, true, true) : GEN_GO(float, true, false))
            : (vec ? GEN_GO(float, false, true) : GEN_GO(float, false, false));
#undef GEN_GO
}

// Pixel ranges: about 512 blocks, at least 32 pixels each, at most 8 MB of
// slices and no more slices than a plan has room for.
static int gen_wgrad_splits(const ConvShape& s) {
  const int bm = s.cout <= 32 ? 32 : 64, bn = s.cout <= 32 ? 128 : 64;
  const long tiles = (long)((s.cout + bm - 1) / bm) * ((s.taps * s.cin + bn - 1) / bn);
  const long E = (long)s.cout * s.taps * s.cin;
  long S = std::min({(512 + tiles - 1) / tiles, (s.pixels() + 31) / 32,
                     std::max(1L, (8L << 20) / (4 * E)), (long)direct_wgrad_splits(s.pixels())});
  const long pps = ((s.pixels() + S - 1) / S + 31) / 32 * 32;
  return (int)((s.pixels() + pps - 1) / pps);
}

size_t conv_gen_wgrad_partial_floats(const ConvShape& s) {
  const int S = gen_wgrad_splits(s);
  return S > 1 ? (size_t)S * s.cout * s.taps * s.cin : 0;
}

template <typename T, bool VEC>
static hipError_t launch_gen_wgrad(int n, const void* const* x, const void* const* dz,
                                   float* const* dw, float* const* partial, const ConvShape& s,
                                   hipStream_t st, ReduceJob* const* defer) {
  const int S = gen_wgrad_splits(s);
  const long P = s.pixels(), E = (long)s.cout * s.taps * s.cin;
  const int pps = (int)(((P + S - 1) / S + 31) / 32 * 32);
  GenWgIo<T> io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    const int q = k < n ? k : 0;
    io.x[k] = (const T*)x[q];
    io.dz[k] = (const T*)dz[q];
    io.part[k] = S > 1 ? partial[q] : dw[q];   // a single range writes the gradient itself
  }
  const bool thin = s.cout <= 32;
  const int bm = thin ? 32 : 64, bn = thin ? 128 : 64;
  const long blocks = (long)n * S * ((s.cout + bm - 1) / bm) * ((s.taps * s.cin + bn - 1) / bn);
  if (blocks >= (1L << 31)) return hipErrorInvalidValue;
  {
    ProfScope ps(thin ? "conv_gen_wgrad<1,4>" : "conv_gen_wgrad<2,2>", 2.0 * n * P * E,
                 n * ((double)sizeof(T) * P * (s.cin + s.cout) + 4.0 * S * E), st);
    if (thin)
      TGP_LAUNCH(ps, (conv_gen_wgrad<T, 1, 4, VEC>), dim3((unsigned)blocks), dim3(256), 0, st, io,
                 (int)P, s.H, s.W, s.cin, s.cout, s.taps, S, pps);
    else
      TGP_LAUNCH(ps, (conv_gen_wgrad<T, 2, 2, VEC>), dim3((unsigned)blocks), dim3(256), 0, st, io,
                 (int)P, s.H, s.W, s.cin, s.cout, s.taps, S, pps);
  }
  const hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{io.part[k], dw[k], E, S};
  return hipSuccess;
}

hipError_t conv_gen_wgrad_launch(int dt, int n, const void* const* x, const void* const* dz,
                                 float* const* dw, float* const* partial, const ConvShape& s,
                                 hipStream_t st, ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup || s.pixels() <= 0) return hipErrorInvalidValue;
  const bool vec = s.cin % 4 == 0 && s.cout % 4 == 0;
  if (dt == 0)
    return vec ? launch_gen_wgrad<bf16_t, true>(n, x, dz, dw, partial, s, st, defer)
               : launch_gen_wgrad<bf16_t, false>(n, x, dz, dw, partial, s, st, defer);
  return vec ? launch_gen_wgrad<float, true>(n, x, dz, dw, partial, s, st, defer)
             : launch_gen_wgrad<float, false>(n, x, dz, dw, partial, s, st, defer);
}

}  // namespace tgpk
