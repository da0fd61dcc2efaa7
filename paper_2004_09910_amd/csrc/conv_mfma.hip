// bf16 implicit-GEMM convolutions on gfx950 MFMA (v_mfma_f32_32x32x16_bf16),
// fp32 accumulation, NHWC activations, KRSC weights.
//
// Forward (and data gradient, which is the same contraction on the rotated,
// transposed weight):  Y^T[co][p] = sum_k W[co][k] * im2col(X)[p][k],
// k = (tap, ci) so that every 64-wide K slice is one filter tap and 64
// contiguous channels: both operands are K-contiguous 128-byte rows that are
// staged into LDS with 16-byte loads.  Each block computes a BN x BM
// (channels x pixels) tile with 4 waves; bias + ReLU + bf16 rounding are fused
// into the epilogue.
//
// Weight gradient:  dW[co][tap][ci] = sum_p dZ[p][co] * X[p + off(tap)][ci],
// K = pixels.  In NHWC both operands are channel-contiguous, so each thread
// loads an 8-pixel x 8-channel block with 16-byte loads and transposes it in
// registers before writing pixel-contiguous rows to LDS.  The pixel range is
// split over grid.z; each split writes its fp32 partial tile and a second
// kernel sums the splits in fixed order (deterministic, no atomics).
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {

// ---------------------------------------------------------------- forward (LDS DMA)

// Sixteen zero bytes in device memory: the source of every im2col chunk that
// falls outside the image (the zero padding), so that all tile loads can be
// direct global -> LDS copies.
__device__ __attribute__((aligned(16))) unsigned int g_zero16[4];

// Implicit-GEMM forward with an NS-stage ring of LDS tiles filled by
// global_load_lds_dwordx4: each wave instruction copies 8 rows of 128 bytes;
// lane l fills physical chunk l & 7 of row l >> 3 with the logical chunk that
// the XOR swizzle puts there.  Loads run NS - 1 K steps ahead of the MFMAs.
// Block index remapped (xcd_remap) so that consecutive pixel tiles, which
// share halo rows and read the same weights, run on the same XCD.

// X2 / Y2 (both null or both set): a second micro-batch of P pixels; the
// grid then holds both micro-batches' tiles, the second half for it.
template <int WCO, int WP, int TM, int TN, int TAPS, int NS>
__global__ __launch_bounds__(WCO * WP * 64) void conv_fwd_dma(
    const bf16_t* __restrict__ X0, const bf16_t* __restrict__ X2, const bf16_t* __restrict__ Wt,
    const float* __restrict__ bias, bf16_t* __restrict__ Y0, bf16_t* __restrict__ Y2, int P,
    int H, int W, int Cin, int Cout, int relu, int co_major) {
  constexpr int NW = WCO * WP;       // waves per block
  constexpr int BN = WCO * TM * 32;  // output channels per block
  constexpr int BM = WP * TN * 32;   // pixels per block
  constexpr int ROWS = BN + BM;
  constexpr int LPS = ROWS / (8 * NW);  // DMA instructions per wave per stage
  static_assert(BN % 64 == 0 && ROWS % (8 * NW) == 0, "tile shape");
  __shared__ u32x4 smem[NS][ROWS * 8];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wco = wave / WP, wp = wave % WP;
  // The grid is (pixel tiles x channel tiles) flattened.  Each XCD gets a
  // contiguous range of it: pixel-tile-major when the activations are the
  // larger operand (an XCD then holds a slice of the image plus all weights
  // in its L2), channel-tile-major when the weights are (a slice of the
  // weights plus the whole activation tile set).
  const int nct = Cout / BN;
  const int per = X2 ? gridDim.x / 2 : gridDim.x;              // blocks per micro-batch
  const int npt = per / nct;
  const int lb0 = xcd_remap(blockIdx.x, gridDim.x);
  const bool g1 = lb0 >= per;                                   // second micro-batch (uniform)
  const int lb = g1 ? lb0 - per : lb0;
  const bf16_t* __restrict__ X = g1 ? X2 : X0;
  bf16_t* __restrict__ Y = g1 ? Y2 : Y0;
  const int p0 = (co_major ? lb % npt : lb / nct) * BM;
  const int co0 = (co_major ? lb / npt : lb % nct) * BN;
  const int K = TAPS * Cin;
  const int cpt = Cin / 64;
  const int nk = TAPS * cpt;
  const int HW = H * W;

  // Source of each row this lane fills, per stage instruction u.
  const bf16_t* src[LPS];
  int ph[LPS], pw[LPS];
  bool pok[LPS];
#pragma unroll
  for (int u = 0; u < LPS; ++u) {
    const int r = (wave + NW * u) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r ^ (r >> 3)) & 7);
    if ((wave + NW * u) * 8 < BN) {
      src[u] = Wt + (long)(co0 + r) * K + c * 8;
      ph[u] = pw[u] = 0;
      pok[u] = true;
    } else {
      const int p = p0 + r - BN;
      pok[u] = p < P;
      const int pp = pok[u] ? p : 0;
      const int rem = pp % HW;
      ph[u] = rem / W;
      pw[u] = rem - ph[u] * W;
      src[u] = X + (long)pp * Cin + c * 8;
    }
  }
  const bf16_t* zero = (const bf16_t*)g_zero16;

  auto issue = [&](int ks, int slot) __attribute__((always_inline)) {
    const int tap = ks / cpt;
    const int c0 = (ks - tap * cpt) * 64;
    const int dr = (TAPS == 9) ? tap / 3 - 1 : 0;
    const int dc = (TAPS == 9) ? tap % 3 - 1 : 0;
    const long shift = ((long)dr * W + dc) * Cin + c0;
#pragma unroll
    for (int u = 0; u < LPS; ++u) {
      const bf16_t* g;
      if ((wave + NW * u) * 8 < BN) {
        g = src[u] + tap * Cin + c0;
      } else {
        const int hh = ph[u] + dr, ww = pw[u] + dc;
        const bool ok = pok[u] && (unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W;
        g = ok ? src[u] + shift : zero;
      }
      __builtin_amdgcn_global_load_lds((const void*)g,
                                       TGP_LDS(&smem[slot][(wave + NW * u) * 64]), 16, 0, 0);
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x16_t{};

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) issue(s, s);
  // this lane's bias values for the epilogue, loaded up front as 16-byte
  // vectors (channels co0 + wco TM 32 + 32 i + 8 g + 4 (lane / 32) + t);
  // loaded one by one at the epilogue they held up every store
  f32x4_t bv[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      bv[i][g] = bias ? *(const f32x4_t*)(bias + co0 + wco * TM * 32 + i * 32 + 8 * g +
                                          4 * (lane >> 5))
                      : f32x4_t{};
  for (int ks = 0; ks < nk; ++ks) {
    const int ahead = min(NS - 2, nk - 1 - ks);
    wait_stages<NS, LPS>(ahead);
    ring_barrier();
    if (ks + NS - 1 < nk) issue(ks + NS - 1, (ks + NS - 1) % NS);
    const u32x4* As = smem[ks % NS];
    const u32x4* Bs = smem[ks % NS] + BN * 8;
    // the fragments of K sub-step kk + 1 are read while the MFMAs of kk run
    bf16x8_t a[2][TM], b[2][TN];
    auto load = [&](int kk, int buf) __attribute__((always_inline)) {
      const int qq = 2 * kk + (lane >> 5);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wco * TM * 32 + i * 32 + (lane & 31);
        a[buf][i] = as_bf16x8(As[row * 8 + swz(row, qq)]);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wp * TN * 32 + j * 32 + (lane & 31);
        b[buf][j] = as_bf16x8(Bs[row * 8 + swz(row, qq)]);
      }
    };
    load(0, 0);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk + 1 < 4) load(kk + 1, (kk + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(a[kk & 1][i], b[kk & 1][j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Epilogue: lanes l and l + 32 hold channels 8 g + 0..3 and 8 g + 4..7
  // of pixel l % 32.  Swapping the halves of groups 2 h and 2 h + 1 across
  // the two half-waves leaves lane l with channels 16 h + 0..7 and lane
  // l + 32 with 16 h + 8..15, so each lane stores 16 contiguous bytes
  // (scattered 8-byte stores cost a memory-pipeline cycle per lane).
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int p = p0 + wp * TN * 32 + j * 32 + (lane & 31);
      unsigned pk[4][2];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[i][j][4 * g + t] + bv[i][g][t];
          if (relu) v[t] = fmaxf(v[t], 0.0f);
        }
        pk[g][0] = f2bf(v[0]) | (f2bf(v[1]) << 16);
        pk[g][1] = f2bf(v[2]) | (f2bf(v[3]) << 16);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(pk[2 * h][r], pk[2 * h + 1][r], false,
                                                           false);
          pk[2 * h][r] = sw[0];
          pk[2 * h + 1][r] = sw[1];
        }
        const int co = co0 + wco * TM * 32 + i * 32 + 16 * h + 8 * (lane >> 5);
        if (p < P)
          *(u32x4*)(Y + (long)p * Cout + co) =
              u32x4{pk[2 * h][0], pk[2 * h][1], pk[2 * h + 1][0], pk[2 * h + 1][1]};
      }
    }
  }
}

// ---------------------------------------------------------------- 1x1, resident weights

// 1x1 convolution y[p][co] = act(sum_ci x[p][ci] w[co][ci] + b[co]) with
// Cout = 256 and Cin = 64 NKS up to 256 (the depthwise/pointwise cells): its K
// is so short that it is bound by reading x and writing y.  So each wave keeps
// its 32 output channels' weights in registers (16 VGPRs per 64 channels), and
// all of LDS is a ring of NS stages of 64 pixels x Cin, three of them in flight:
// 96 KiB a CU.  The loads are issued from inline assembly (the compiler would
// wait for all of them before every LDS read), and in the steady state the wait
// counts the stores of the tiles between, so that it does not wait for those
// either.  Measured at 256 -> 256, 56 x 56 x 4, sixteen micro-batches: weights
// in LDS and four stages of 64 pixels x 64 channels 61 us, this 48.  Wave w
// computes output channels 32 w .. 32 w + 31 of the tile's 64 pixels (two 32 x
// 32 MFMA tiles), so every pixel row is read once.  The K order (16-channel MFMA
// steps, increasing channel) is the other 1x1 kernels', so they give the same
// bits.  Blocks are persistent over the tiles of all ng micro-batches of the
// launch (each of P pixels, micro-batch k's tiles after those of k - 1).
struct Mb1x1 {
  const bf16_t* x[kMaxGroup];
  bf16_t* y[kMaxGroup];
};
template <int NKS, int NS>
__global__ __launch_bounds__(512) void conv1x1_res(Mb1x1 io, int ng,
                                                   const bf16_t* __restrict__ Wt,
                                                   const float* __restrict__ bias, int P, int relu) {
  constexpr int COUT = 256, BM = 64, CIN = 64 * NKS;
  constexpr int SB = BM * CIN * 2;                              // stage bytes
  static_assert(NS * SB <= 160 * 1024, "LDS ring");
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * SB];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T1 = (P + BM - 1) / BM;                             // tiles per micro-batch
  const int T = ng * T1;
  const int G = gridDim.x;
  const int lb = xcd_remap(blockIdx.x, G);
  const int n_mine = lb < T ? (T - lb + G - 1) / G : 0;

  // This wave's weights: fragment k holds channels 16 k + 8 (lane / 32) .. + 7.
  bf16x8_t wf[4 * NKS];
#pragma unroll
  for (int k = 0; k < 4 * NKS; ++k)
    wf[k] = as_bf16x8(
        *(const u32x4*)(Wt + (long)(32 * wave + (lane & 31)) * CIN + 16 * k + 8 * (lane >> 5)));
  // and bias values (channels 32 wave + 8 g + 4 (lane / 32) + t)
  f32x4_t bv[4];
#pragma unroll
  for (int g = 0; g < 4; ++g)
    bv[g] = bias ? *(const f32x4_t*)(bias + 32 * wave + 8 * g + 4 * (lane >> 5)) : f32x4_t{};

  // DMA: instruction u of this wave fills rows 8 wave .. + 7 (128 bytes, chunks
  // XOR-swizzled) of the stage's 64-channel block u; pixels past P read zeros.
  const int xr = wave * 8 + (lane >> 3);
  const int xoff = xr * CIN * 2 + (((lane & 7) ^ ((xr ^ (xr >> 3)) & 7)) << 4);
  auto issue = [&](int it) __attribute__((always_inline)) {
    const int tt = lb + it * G;
    const int gi = tt / T1;                                     // micro-batch (uniform)
    const u32x4 rx = make_rsrc(pickg(io.x, gi), P * CIN * 2);
    const int p0 = (tt - gi * T1) * BM;
#pragma unroll
    for (int u = 0; u < NKS; ++u)
      dma16(rx, TGP_LDS(ring + (it % NS) * SB + u * BM * 128 + wave * 1024), xoff + u * 128,
            p0 * CIN * 2);
  };
#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < n_mine) issue(k);

  const bool whole = P % BM == 0;                               // every tile stores 4 times a wave
  for (int it = 0; it < n_mine; ++it) {
    const int tt = lb + it * G;
    const int gi = tt / T1;
    bf16_t* __restrict__ Y = pickg(io.y, gi);
    const int p0 = (tt - gi * T1) * BM;
    f32x16_t acc[2] = {f32x16_t{}, f32x16_t{}};
    // Stage `it` is in once at most what was issued after it is pending: the
    // NS - 2 stages after it and, from the NS - 1st tile on, the stores of the
    // NS - 1 tiles before this one.
    if (whole && it >= NS - 1 && it + NS - 2 < n_mine)
      wait_vmcnt<(NS - 2) * NKS + (NS - 1) * 4>();
    else
      wait_stages<NS, NKS>(min(NS - 2, n_mine - 1 - it));
    ring_barrier();
    if (it + NS - 1 < n_mine) issue(it + NS - 1);
    const u32x4* Bs = (const u32x4*)(ring + (it % NS) * SB);
    bf16x8_t b[2][2];
    auto load = [&](int k, int buf) __attribute__((always_inline)) {
      const int qq = 2 * (k & 3) + (lane >> 5);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int rb = 32 * j + (lane & 31);
        b[buf][j] = as_bf16x8(Bs[(k >> 2) * BM * 8 + rb * 8 + swz(rb, qq)]);
      }
    };
    load(0, 0);
#pragma unroll
    for (int k = 0; k < 4 * NKS; ++k) {
      if (k + 1 < 4 * NKS) load(k + 1, (k + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = mfma32(wf[k], b[k & 1][j], acc[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // Epilogue: lanes l and l + 32 hold channels 8 g + 0..3 and 8 g + 4..7
    // of pixel l % 32; swapping the halves of groups 2 h and 2 h + 1 across
    // the half-waves leaves each lane 8 consecutive channels, one 16-byte
    // store.
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int p = p0 + 32 * j + (lane & 31);
      unsigned pk[4][2];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[j][4 * g + t] + bv[g][t];
          if (relu) v[t] = fmaxf(v[t], 0.0f);
        }
        pk[g][0] = f2bf(v[0]) | (f2bf(v[1]) << 16);
        pk[g][1] = f2bf(v[2]) | (f2bf(v[3]) << 16);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(pk[2 * h][r], pk[2 * h + 1][r], false,
                                                           false);
          pk[2 * h][r] = sw[0];
          pk[2 * h + 1][r] = sw[1];
        }
        if (p < P)
          *(u32x4*)(Y + (long)p * COUT + 32 * wave + 16 * h + 8 * (lane >> 5)) =
              u32x4{pk[2 * h][0], pk[2 * h][1], pk[2 * h + 1][0], pk[2 * h + 1][1]};
      }
    }
  }
}

// ---------------------------------------------------------------- wgrad

// 8x8 transpose of bfloat16: in[j] holds 8 channels of pixel j; out[c] gets
// 8 pixels of channel c.
__device__ __forceinline__ void transpose8x8(const u32x4 (&in)[8], u32x4 (&out)[8]) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    uint32_t d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t lo = in[2 * e][c >> 1];
      uint32_t hi = in[2 * e + 1][c >> 1];
      d[e] = (c & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
    }
    out[c] = u32x4{d[0], d[1], d[2], d[3]};
  }
}

// The ng micro-batches of one launch: micro-batch k's blocks form the k-th
// of ng equal parts of the grid.
struct MbWg {
  const bf16_t* x[kMaxGroup];
  const bf16_t* dz[kMaxGroup];
  float* part[kMaxGroup];
};
template <int WM, int WN, int TM, int TN, int TAPS>
__global__ __launch_bounds__(256) void conv_wgrad_mfma(MbWg io, int ng, int P, int H, int W,
                                                       int Cin, int Cout, int pix_per_split) {
  static_assert(WM * WN == 4, "4 waves");
  constexpr int BMc = WM * TM * 32;  // output channels (co) per block
  constexpr int BNc = WN * TN * 32;  // input channels (ci) per block
  constexpr int BK = 64;             // pixels per K step
  static_assert(BMc + BNc <= 256, "one 8x8 block per thread");
  __shared__ u32x4 smem[2][(BMc + BNc) * 8];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int ncb = Cin / BNc;
  // 1-D grid of (split, tap, ci tile, co tile), split slowest.  The
  // dispatcher deals blocks round-robin over the 8 XCDs; remapped, each XCD
  // runs a contiguous range of splits with all their tiles, so the pixel rows
  // of X and dZ a split reads are fetched into one L2 only.
  const int T = TAPS * ncb * (Cout / BMc);
  const int per = gridDim.x / ng;                               // blocks per micro-batch
  const int lb0 = xcd_remap(blockIdx.x, gridDim.x);
  const int gi = lb0 / per;                                     // micro-batch (uniform)
  const int lb = lb0 - gi * per;
  const bf16_t* __restrict__ X = pickg(io.x, gi);
  const bf16_t* __restrict__ dZ = pickg(io.dz, gi);
  float* __restrict__ part = pickg(io.part, gi);
  const int split = lb / T;
  const int t = lb - split * T;
  const int tx = t % (TAPS * ncb);
  const int tap = tx / ncb;
  const int ci0 = (tx - tap * ncb) * BNc;
  const int co0 = (t / (TAPS * ncb)) * BMc;
  const int ps = split * pix_per_split;
  const int pe = min(P, ps + pix_per_split);
  const int nk = (pe - ps + BK - 1) / BK;
  const int dr = (TAPS == 9) ? tap / 3 - 1 : 0;
  const int dc = (TAPS == 9) ? tap % 3 - 1 : 0;

  // Load role: threads [0, BMc) load dZ blocks, [BMc, BMc+BNc) load X blocks.
  const bool isA = tid < BMc;
  const bool active = tid < BMc + BNc;
  const int t2 = isA ? tid : tid - BMc;
  const int nchunk = isA ? BMc / 8 : BNc / 8;
  const int cc = t2 % nchunk;      // 8-channel chunk
  const int pc = t2 / nchunk;      // 8-pixel chunk within the K step (0..7)

  u32x4 v[8];
  auto gload = [&](int ks) {
    int pbase = ps + ks * BK + pc * 8;
    if (!active) return;
    if (isA) {
      const bf16_t* src = dZ + (long)pbase * Cout + co0 + cc * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = (pbase + j < pe) ? *(const u32x4*)(src + (long)j * Cout) : u32x4{0, 0, 0, 0};
    } else {
      int HW = H * W;
      int pp = pbase < P ? pbase : 0;
      int rem = pp % HW;
      int h = rem / W, w = rem - h * W;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        int hh = h + dr, ww = w + dc;
        bool ok = (pbase + j < pe) && (unsigned)hh < (unsigned)H && (unsigned)ww < (unsigned)W;
        v[j] = ok ? *(const u32x4*)(X + ((long)(pbase + j) + (long)dr * W + dc) * Cin + ci0 + cc * 8)
                  : u32x4{0, 0, 0, 0};
        if (++w == W) { w = 0; if (++h == H) h = 0; }
      }
    }
  };
  auto lstore = [&](int buf) {
    if (!active) return;
    u32x4 o[8];
    transpose8x8(v, o);
    u32x4* dst = smem[buf] + (isA ? 0 : BMc * 8);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      int row = cc * 8 + c;
      dst[row * 8 + swz(row, pc)] = o[c];
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x16_t{};

  if (nk > 0) {
    gload(0);
    lstore(0);
  }
  __syncthreads();
  for (int ks = 0; ks < nk; ++ks) {
    const int buf = ks & 1;
    if (ks + 1 < nk) gload(ks + 1);
    const u32x4* As = smem[buf];
    const u32x4* Bs = smem[buf] + BMc * 8;
    // the fragments of K sub-step kk + 1 are read while the MFMAs of kk run
    bf16x8_t a[2][TM], b[2][TN];
    auto load = [&](int kk, int fb) __attribute__((always_inline)) {
      const int qq = 2 * kk + (lane >> 5);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * TM * 32 + i * 32 + (lane & 31);
        a[fb][i] = as_bf16x8(As[row * 8 + swz(row, qq)]);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * TN * 32 + j * 32 + (lane & 31);
        b[fb][j] = as_bf16x8(Bs[row * 8 + swz(row, qq)]);
      }
    };
    load(0, 0);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      if (kk + 1 < BK / 16) load(kk + 1, (kk + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(a[kk & 1][i], b[kk & 1][j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (ks + 1 < nk) lstore(buf ^ 1);
    __syncthreads();
  }

  float* out = part + (long)split * Cout * TAPS * Cin;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      int ci = ci0 + wn * TN * 32 + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int co = co0 + wm * TM * 32 + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        out[((long)co * TAPS + tap) * Cin + ci] = acc[i][j][r];
      }
    }
}

// out[e] = sum_{s < S} part[s][e] in a fixed order: a block of 1024 threads
// covers C4 float4 columns with LANES = 1024 / C4 split lanes; lane l sums
// s = l, l + LANES, ... in ascending order, then lanes 0 .. LANES - 1 are
// added in order.  (C4, LANES) is a function of S only, so the order is a
// function of the shape.  E must be a multiple of 4.
// Blocks from nblk1 on run a second, independent sum (part2, out2, E2, S2)
// in the same launch.
template <int C4>
__global__ __launch_bounds__(1024) void splitk_reduce(const float* __restrict__ part,
                                                      float* __restrict__ out, long E, int S,
                                                      const float* __restrict__ part2,
                                                      float* __restrict__ out2, long E2, int S2,
                                                      int nblk1) {
  constexpr int LANES = 1024 / C4;
  __shared__ float4 red[LANES][C4];
  int bx = blockIdx.x;
  if (bx >= nblk1) {   // block-uniform
    bx -= nblk1;
    part = part2; out = out2; E = E2; S = S2;
  }
  const int col = threadIdx.x % C4, lane = threadIdx.x / C4;
  const long e4 = ((long)bx * C4 + col) * 4;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (e4 < E) {
    int k = lane;
    // eight independent loads in flight per step
    for (; k + 7 * LANES < S; k += 8 * LANES) {
      float4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = *(const float4*)(part + (long)(k + u * LANES) * E + e4);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        acc.x += t[u].x; acc.y += t[u].y; acc.z += t[u].z; acc.w += t[u].w;
      }
    }
    for (; k < S; k += LANES) {
      const float4 t = *(const float4*)(part + (long)k * E + e4);
      acc.x += t.x; acc.y += t.y; acc.z += t.z; acc.w += t.w;
    }
  }
  red[lane][col] = acc;
  __syncthreads();
  if (lane == 0 && e4 < E) {
    float4 r = red[0][col];
    for (int l = 1; l < LANES; ++l) {
      const float4 t = red[l][col];
      r.x += t.x; r.y += t.y; r.z += t.z; r.w += t.w;
    }
    *(float4*)(out + e4) = r;
  }
}

// The same sum of any E (the bias of a one-channel head, a group's bias
// sums): a block takes C = 2^lc columns (up to 64), 256 / C split lanes added
// in a fixed tree (one thread a column took 10.7 us for 144 splits of one, this 4.0).
struct SumGroup {
  const float* part[kMaxGroup];
  float* out[kMaxGroup];
};
__global__ __launch_bounds__(256) void splitk_reduce_scalar(SumGroup io, long E, int S, int lc) {
  __shared__ float red[256];
  const float* __restrict__ part = pickg(io.part, blockIdx.y);
  float* __restrict__ out = pickg(io.out, blockIdx.y);
  const int C = 1 << lc, col = threadIdx.x & (C - 1), lane = threadIdx.x >> lc;
  const long e = (long)blockIdx.x * C + col;
  float acc = 0.f;
  if (e < E)
    for (int k = lane; k < S; k += 256 >> lc) acc += part[(long)k * E + e];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 128 >> lc; h > 0; h >>= 1) {
    if (lane < h) red[threadIdx.x] += red[threadIdx.x + (h << lc)];
    __syncthreads();
  }
  if (lane == 0 && e < E) out[e] = red[threadIdx.x];
}

// wt[ci][tap'][co] = w[co][taps-1-tap'][ci]: the data gradient of a
// cross-correlation is a cross-correlation with the 180-degree rotated,
// channel-transposed filter.  A batch of tensors in one launch: blocks
// blk0[k] .. blk0[k + 1] - 1 serve tensor k.
template <typename T>
__global__ void wtransform_batch_kernel(WtBatch b) {
  int k = 0;
  while (k + 1 < b.count && (int)blockIdx.x >= b.blk0[k + 1]) ++k;
  const long e = (long)(blockIdx.x - b.blk0[k]) * 256 + threadIdx.x;
  const int cout = b.cout[k], cin = b.cin[k], taps = b.taps[k];
  if (e >= (long)cout * cin * taps) return;
  const int co = e % cout;
  const long r = e / cout;
  const int tp = r % taps;
  const int ci = r / taps;
  ((T*)b.wt[k])[e] = ((const T*)b.w[k])[((long)co * taps + (taps - 1 - tp)) * cin + ci];
}

struct WgradPlan {
  int S, pix_per_split;
};

// Split count for the weight gradient: enough blocks to fill the chip
// (~512), at least 256 pixels per split, and at most ~8 MB of fp32 partials
// (their write + fixed-order re-read otherwise costs more than the extra
// parallelism gains).
template <int TM, int TN>
WgradPlan wgrad_plan(long P, int tiles, long E) {
  const int BK = 64;
  int S = cdiv(512, tiles);
  int maxS = cdiv(P, 256);
  if (S > maxS) S = maxS;
  long cap = (8L << 20) / (4 * E);
  if (S > cap) S = (int)cap;
  if (S < 1) S = 1;
  int pps = cdiv(cdiv(P, S), BK) * BK;
  S = cdiv(P, pps);
  return {S, pps};
}

}  // namespace

// ---------------------------------------------------------------- dispatch

bool mfma_conv_ok(int dt, int cin, int cout) {
  return dt == 0 && cin % 64 == 0 && cout % 64 == 0;
}
// Shapes conv_forward_mfma takes: those, and the layers of the kernels for
// any multiple of 8 channels.
bool mfma_fwd_ok(int dt, const ConvShape& s) {
  return mfma_conv_ok(dt, s.cin, s.cout) || (dt == 0 && (conv_tile_ok(s) || conv1x1_tile_ok(s)));
}

// Forward tile configurations.  A configuration is chosen per shape by
// fwd_config() (a pure function of the shape, so recomputation reuses the
// exact same kernel); g_fwd_variant > 0 forces one for measurement sweeps.
int g_fwd_variant = 0;
int g_fwd_order = -1;   // -1: by operand size; 0/1 forced (measurement only)

template <int WCO, int WP, int TM, int TN, int NS>
hipError_t launch_fwd_dma(const char* name9, const char* name1, const bf16_t* X, const bf16_t* Wt,
                          const float* b, bf16_t* Y, long P, const ConvShape& s, int relu,
                          hipStream_t st, const bf16_t* X2 = nullptr, bf16_t* Y2 = nullptr) {
  const char* name = s.taps == 9 ? name9 : name1;
  constexpr int BN = WCO * TM * 32, BM = WP * TN * 32;
  if (s.cout % BN || (X2 == nullptr) != (Y2 == nullptr)) return hipErrorInvalidValue;
  const int ng = X2 ? 2 : 1;
  dim3 grid(ng * cdiv(P, BM) * (s.cout / BN));
  double flops = 2.0 * ng * P * s.cout * s.taps * s.cin;
  double bytes = 2.0 * ((double)ng * P * s.cin + (double)s.cout * s.taps * s.cin +
                        (double)ng * P * s.cout);
  ProfScope ps(name, flops, bytes, st);
  const double xbytes = 2.0 * P * s.cin, wbytes = 2.0 * s.cout * s.taps * s.cin;
  const int co_major = g_fwd_order >= 0 ? g_fwd_order : (wbytes > xbytes ? 1 : 0);
  if (s.taps == 9)
    TGP_LAUNCH(ps, (conv_fwd_dma<WCO, WP, TM, TN, 9, NS>), grid, dim3(WCO * WP * 64), 0, st, X,
                       X2, Wt, b, Y, Y2, (int)P, s.H, s.W, s.cin, s.cout, relu, co_major);
  else
    TGP_LAUNCH(ps, (conv_fwd_dma<WCO, WP, TM, TN, 1, NS>), grid, dim3(WCO * WP * 64), 0, st, X,
                       X2, Wt, b, Y, Y2, (int)P, s.H, s.W, s.cin, s.cout, relu, co_major);
  return launch_status();
}

#define TGP_FWD_CFG(WCO, WP, TM, TN, NS)                                                        \
  launch_fwd_dma<WCO, WP, TM, TN, NS>("conv_fwd_dma<" #WCO "," #WP "," #TM "," #TN ",9," #NS ">", \
                                      "conv_fwd_dma<" #WCO "," #WP "," #TM "," #TN ",1," #NS ">", \
                                      X, Wt, b, Y, P, s, relu, st, X2, Y2)

int g_fwd_split = 0;   // > 0 forces the shares of a sum (measurement only)
// Measurement only: bit 2 allows the row-blocked weight gradient, bit 3 the
// nine-tap row kernel.
int g_rowtile_mask = 15;

struct FwdPlan {
  int cfg;   // 100+: per-tap (150: 1x1 with resident weights); 300+: row-tiled; 400+:
             // whole-row; 500+: rectangular tiles; 600+: 1x1 tiles
  int S;     // shares of the sum (500)
};

// The resident-weight 1x1 kernel's shapes and its launch.
static bool conv1x1_res_ok(const ConvShape& s) {
  return s.cout == 256 && s.cin % 64 == 0 && s.cin <= 256 && conv1x1_tile_ok(s);
}

// n micro-batches x[k] -> y[k] in one launch.
static hipError_t launch_1x1_res(int n, const void* const* x, const bf16_t* Wt, const float* b,
                                 void* const* y, const ConvShape& s, int relu, hipStream_t st) {
  if (!conv1x1_res_ok(s) || n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const long P = s.pixels();
  if (P > (1L << 30)) return hipErrorInvalidValue;              // pixel index is an int
  Mb1x1 io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.y[k] = (bf16_t*)y[k < n ? k : 0];
  }
  const long T = n * ((P + 63) / 64);
  const int G = (int)(T < 256 ? T : 256);
  ProfScope ps("conv1x1_res", 2.0 * n * P * s.cout * s.cin,
               2.0 * ((double)n * P * (s.cin + s.cout) + (double)s.cout * s.cin), st);
  switch (s.cin / 64) {
    case 1: TGP_LAUNCH(ps, (conv1x1_res<1, 8>), dim3(G), dim3(512), 0, st, io, n, Wt, b, (int)P, relu); break;
    case 2: TGP_LAUNCH(ps, (conv1x1_res<2, 8>), dim3(G), dim3(512), 0, st, io, n, Wt, b, (int)P, relu); break;
    case 3: TGP_LAUNCH(ps, (conv1x1_res<3, 5>), dim3(G), dim3(512), 0, st, io, n, Wt, b, (int)P, relu); break;
    default: TGP_LAUNCH(ps, (conv1x1_res<4, 4>), dim3(G), dim3(512), 0, st, io, n, Wt, b, (int)P, relu);
  }
  return launch_status();
}

// Pure function of one micro-batch's shape, plus the measurement overrides: the
// kernel family and the split count fix the K summation order, so a
// recomputation and a launch over several micro-batches give the same bits.
// Both depend on the per-sample shape alone (split counts use a nominal
// micro-batch of 4 samples), which keeps a sample's output bit-identical
// whatever the micro-batch size, with one exception: images from 24 x 24 to below
// 48 x 48 of the whole-row kernel's widths, where that kernel needs 48 tiles of
// the micro-batch and adds each sum in one chain, while the rectangular tiles
// that run otherwise split deep sums (512 channels at 24 x 24: one sample in
// shares, two or more in one chain).  Making that choice per sample cost single
// samples up to 19% (896 -> 256 at 24 x 24) or groups of them the whole rows.
FwdPlan fwd_plan(const ConvShape& s) {
  FwdPlan pl{0, 1};
  if (s.cin % 64 || s.cout % 64) {   // the kernels that take any multiple of 8
    pl.cfg = s.taps == 9 ? 500 : 600;
    if (g_fwd_variant >= pl.cfg && g_fwd_variant < pl.cfg + 100) pl.cfg = g_fwd_variant;
    return pl;
  }
  // The nine-tap whole-row kernel on images of 48 x 48 and up of the widths it
  // is built for, and from 24 x 24 where one micro-batch gives it at least 48
  // tiles; the rectangular tiles for every other 3x3 layer (us, forward + data
  // gradient with the transform of its weights, against the kernels these
  // shapes had: 64 at 224 x 224 x 1 22 / 44, x 16 185 / 285; 256 at 56 x 56 x 8 75
  // / 141, x 1 29 / 61; 256 at 28 x 28 x 32 79 / 237; 64 at 14 x 14 x 2 12 / 44).
  const bool k3 = s.taps == 9;
  const long hw = (long)s.H * s.W;
  if (k3 && (hw >= 48 * 48 || (hw >= 24 * 24 && conv_rows32_tiles(s) >= 48)) &&
      (g_rowtile_mask >> 3 & 1) && conv_rows32_ok(s)) {
    pl.cfg = 400;  // whole-row tiles, nine taps per stage, 32x32x16
  } else if (conv1x1_res_ok(s)) {
    pl.cfg = 150;  // 1x1, weights in registers
  } else if (conv_tile_ok(s)) {
    pl.cfg = 500;  // rectangular tiles
  } else if (conv1x1_tile_ok(s)) {
    pl.cfg = 600;  // 1x1 tiles
  } else {
    pl.cfg = 100;
  }
  if (g_fwd_variant > 0) pl.cfg = g_fwd_variant;
  if (pl.cfg == 150 && !conv1x1_res_ok(s)) pl.cfg = 100;
  if (pl.cfg >= 500) {
    if (pl.cfg >= 600 ? !conv1x1_tile_ok(s) : !conv_tile_ok(s)) pl.cfg = 100;
    if (pl.cfg < 600)
      pl.S = g_fwd_split > 0 && s.cin / 16 % g_fwd_split == 0 ? g_fwd_split : conv_tile_split(s);
    return pl;
  }
  if (pl.cfg >= 400) {
    g_rows32_cfg = pl.cfg >= 401 ? pl.cfg - 401 : -1;
    if (!conv_rows32_ok(s)) pl.cfg = 100;
    g_rows32_cfg = -1;
    return pl;
  }
  if (pl.cfg >= 300) {
    if (!conv_rowtile_ok(s)) pl.cfg = 100;
    return pl;
  }
  if (pl.cfg < 100 || (pl.cfg >= 200 && pl.cfg < 300)) pl.cfg = 100;   // no such kernel
  return pl;
}

// A launch of the whole-row kernel's shapes that is too small for it: its tiles
// are whole rows, so few samples leave CUs idle, where the rectangular tiles can
// be smaller.  Both sum over (chunk, tap, channel), so the choice does not
// change a bit.  The line is where a launch has 2304 tiles of 32 pixels x 32
// channels: up to and at it with up to 128 input channels, below it with more,
// whose stages are many.  At it (us, forward, rectangular / rows): 128 at 96 x 96 x
// 2 13.6 / 15.9, 64 at 192 x 192 x 1 10.2 / 14.2; 256 at 48 x 48 x 4 20.4 / 20.2, 512
// at 24 x 24 x 8 37.1 / 34.6, 256 -> 64 at 96 x 96 x 4 30.3 / 23.2, 2048 -> 256 at 24
// x 24 x 16 138 / 123.  Past it: 128 at 96 x 96 x 4 22.3 / 19.8.
static bool tile_instead(const FwdPlan& pl, const ConvShape& s, int n) {
  return pl.cfg == 400 && g_fwd_variant == 0 &&
         n * s.pixels() * s.cout < 2304L * 1024 + (s.cin <= 128 ? 1 : 0) && conv_tile_ok(s);
}

// The rectangular-tile kernel (500 ..) or the 1x1 tile kernel (600 ..), in the
// configuration a forced plan names.
static hipError_t launch_tile_cfg(const FwdPlan& pl, int n, const void* const* x, const void* w,
                                  const float* b, void* const* y, const ConvShape& s, int relu,
                                  bool dg, float* const* part, size_t part_cap, hipStream_t st) {
  const int cfg = pl.cfg;
  if (s.taps == 1) {
    g_1x1_cfg = cfg >= 601 ? cfg - 601 : -1;
    const hipError_t e = conv_forward_1x1(n, x, w, b, y, s, relu, dg, st);
    g_1x1_cfg = -1;
    return e;
  }
  if (pl.S > 1 && (size_t)pl.S * s.pixels() * s.cout > part_cap) return hipErrorInvalidValue;
  g_tile_cfg = cfg >= 501 ? cfg - 501 : -1;
  const hipError_t e = conv_forward_tile(n, x, w, b, y, s, relu, dg, pl.S, part, st);
  g_tile_cfg = -1;
  return e;
}

// Whether a shape's data gradient (t: its transposed shape) over n micro-batches
// (and then over any fewer) runs on a kernel that reads the forward weights, and
// that launch (also where a forced plan names another kernel but no transformed
// weights were planned for).
bool conv_dgrad_tile_now(const ConvShape& t, int n) {
  const FwdPlan pl = fwd_plan(t);
  return pl.cfg >= 500 || tile_instead(pl, t, n);
}
hipError_t conv_dgrad_tile(int n, const void* const* dz, const void* w, void* const* dx,
                           const ConvShape& t, float* const* part, size_t part_cap,
                           hipStream_t st) {
  FwdPlan pl = fwd_plan(t);
  if (pl.cfg < 500) pl = FwdPlan{t.taps == 9 ? 500 : 600, 1};
  return launch_tile_cfg(pl, n, dz, w, nullptr, dx, t, 0, true, part, part_cap, st);
}

size_t conv_forward_partial_floats(int dt, const ConvShape& s) {
  if (!mfma_fwd_ok(dt, s)) return 0;
  FwdPlan pl = fwd_plan(s);
  return pl.S > 1 ? (size_t)pl.S * s.pixels() * s.cout : 0;
}

hipError_t conv_forward_mfma(const void* x, const void* w, const float* b, void* y,
                             const ConvShape& s, int relu, float* part, size_t part_cap,
                             hipStream_t st) {
  long P = s.pixels();
  const bf16_t* X = (const bf16_t*)x;
  const bf16_t* Wt = (const bf16_t*)w;
  bf16_t* Y = (bf16_t*)y;
  const bf16_t* X2 = nullptr;   // per-tap configurations: one micro-batch
  bf16_t* Y2 = nullptr;
  const FwdPlan pl = fwd_plan(s);
  if (tile_instead(pl, s, 1))
    return launch_tile_cfg(FwdPlan{500, 1}, 1, &x, w, b, &y, s, relu, false, nullptr, 0, st);
  if (pl.cfg == 150) return launch_1x1_res(1, &x, Wt, b, &y, s, relu, st);
  if (pl.cfg >= 500)
    return launch_tile_cfg(pl, 1, &x, w, b, &y, s, relu, false, &part, part_cap, st);
  if (pl.cfg >= 400) {
    g_rows32_cfg = pl.cfg >= 401 ? pl.cfg - 401 : -1;
    const hipError_t e = conv_forward_rows32(1, &x, w, b, &y, s, relu, st);
    g_rows32_cfg = -1;
    return e;
  }
  if (pl.cfg >= 300) {
    g_rowtile_cfg = pl.cfg >= 301 ? pl.cfg - 301 : -1;
    const hipError_t e = conv_forward_rowtile(x, w, b, y, s, relu, st);
    g_rowtile_cfg = -1;
    return e;
  }
  // per-tap kernel (1x1 convolutions, and reference configurations)
  const int v = pl.cfg >= 100 ? pl.cfg - 100 : 0;
  switch (v) {
    case 1: return TGP_FWD_CFG(2, 2, 1, 1, 2);          // 64 x 64, 4 waves
    case 2: return TGP_FWD_CFG(2, 4, 1, 1, 2);          // 64 x 128, 8 waves
    default: return P >= 32768 && s.cout <= 128 ? TGP_FWD_CFG(2, 4, 1, 1, 2)
                                                 : TGP_FWD_CFG(2, 2, 1, 1, 2);
  }
}

hipError_t weight_transform_batch(int dt, WtBatch b, hipStream_t st) {
  if (b.count < 0 || b.count > kMaxWt) return hipErrorInvalidValue;
  long blocks = 0;
  double bytes = 0;
  for (int k = 0; k < b.count; ++k) {
    const long n = (long)b.cout[k] * b.cin[k] * b.taps[k];
    if (n <= 0) return hipErrorInvalidValue;
    b.blk0[k] = (int)blocks;
    blocks += cdiv(n, 256);
    bytes += 2.0 * n * (dt == 0 ? 2 : 4);
  }
  if (b.count == 0) return hipSuccess;
  if (blocks >= (1L << 31)) return hipErrorInvalidValue;
  ProfScope ps("wtransform", 0.0, bytes, st);
  if (dt == 0)
    TGP_LAUNCH(ps, wtransform_batch_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, st, b);
  else
    TGP_LAUNCH(ps, wtransform_batch_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, b);
  return launch_status();
}

// Bit 2 of g_rowtile_mask selects the row-blocked weight-gradient kernel.
static bool use_wgrad_rows(const ConvShape& s) {
  return (g_rowtile_mask >> 2 & 1) && wgrad_rows_ok(s);
}

// Split count of the general weight gradients (per-tap, or the pixel ranges of
// channels that are no multiples of 64): what a plan's slices may take.
int wgrad_general_splits(const ConvShape& s) {
  if (s.cin % 64 || s.cout % 64) return direct_wgrad_splits(s.pixels());
  const int t = s.cin % 128 == 0 && s.cout % 128 == 0 ? 128 : 64;
  return wgrad_plan<2, 2>(s.pixels(), s.taps * (s.cin / t) * (s.cout / t),
                          (long)s.cout * s.taps * s.cin).S;
}

int wgrad_room_splits(int dt, const ConvShape& s) {
  if (dt != 0 || s.cin % 64 || s.cout % 64) return direct_wgrad_splits(s.pixels());
  if (!use_wgrad_rows(s)) return wgrad_general_splits(s);
  const size_t S = wgrad_rows_partial_floats(s) / ((size_t)s.cout * s.taps * s.cin);
  return S > 1 ? (int)S : 1;
}

// 3x3 layers of no fixed width: the rectangular-stage kernel.  Where the
// per-tap kernel can run too (channels in multiples of 64), small layers and
// those whose rows fill the stages badly stay with it.
//  - Its many short blocks start and end sooner, so the lines for one micro-batch
//    a launch and for several lie apart, and one has to serve both (a group gives
//    the bits of single launches): 48 thousand pixel x item products.  Rectangular /
//    per-tap, us with the sum, for one, two and four micro-batches a launch: 128 at
//    56 x 56 x 4 33 / 29, 37 / 33, 39 / 45; 128 -> 192 at 45 x 61 x 3 31 / 28, 35 / 35,
//    40 / 69; x 6 47 / 45, 50 / 55, 55 / 110; 64 at 56 x 56 x 4 23 / 17, 26 / 19, 29 / 30.
//  - A stage's rows are padded to 8 pixels and its k steps to 16: where more than
//    35% of what is multiplied is padding the per-tap kernel wins (384 -> 512 at 15
//    x 10 x 16 96 / 57, 512 -> 256 at 100 x 4 x 4 75 / 43).
// Over 700 random shapes (8 to 500 thousand products) the choice is 3.2%, 1.7% and
// 3.9% from the faster of the two for one, two and four micro-batches a launch;
// the per-tap kernel alone is 4%, 8% and 40% from it.
//  - Below 256 pixels a plan has room for one K range, so an item's stages, one or
//    more a sample, run as a chain: three and more samples of channels that the
//    per-tap kernel does not take go to the pixel-tiled kernel, except where many
//    items multiply long enough for the faster unit to win (rectangular / pixel
//    tiles, us: 24 -> 16 at 6 x 4 x 10 27 / 9; 552 -> 520 at 6 x 3 x 13 40 / 61).  Over
//    250 shapes 1.5 times faster in the mean, three up to 1.19 times slower.
static bool wgrad_chain(const ConvShape& s) {
  return (s.cin % 64 || s.cout % 64) && s.pixels() < 256 && s.nb >= 3 &&
         s.pixels() * ((s.cin + 63) / 64) * ((s.cout + 63) / 64) <= 4096;
}
static bool use_wgrad_tile(const ConvShape& s) {
  if (!wgrad_tile_ok(s) || wgrad_chain(s)) return false;
  return s.cin % 64 || s.cout % 64 ||
         (s.pixels() * (s.cin / 64) * (s.cout / 64) >= 48 * 1024 && wgrad_tile_fill(s) >= 0.65);
}
// Shapes conv_wgrad_mfma takes.
bool mfma_wgrad_ok(int dt, const ConvShape& s) {
  return mfma_conv_ok(dt, s.cin, s.cout) || (dt == 0 && ((wgrad_tile_ok(s) && !wgrad_chain(s)) || wgrad1x1_tile_ok(s)));
}

size_t wgrad_mfma_partial_floats(const ConvShape& s) {
  if (use_wgrad_rows(s)) return wgrad_rows_partial_floats(s);
  if (use_wgrad_tile(s)) return wgrad_tile_partial_floats(s);
  if (wgrad1x1_tile_ok(s)) return wgrad1x1_tile_partial_floats(s);
  int tiles = s.taps * (s.cin / 64) * (s.cout / 64);
  if (s.cin % 128 == 0 && s.cout % 128 == 0) tiles = s.taps * (s.cin / 128) * (s.cout / 128);
  long E = (long)s.cout * s.taps * s.cin;
  WgradPlan pl = wgrad_plan<2, 2>(s.pixels(), tiles, E);
  return (size_t)pl.S * E;
}

// The per-tap weight gradient of n micro-batches in one grid; the split plan
// is the single micro-batch's either way.  Where the plan has one split,
// part[k] is set to dw[k] (the kernel writes the gradient itself).
static hipError_t launch_wgrad_mfma(int n, const void* const* x, const void* const* dz,
                                    float* const* dw, float** part, const ConvShape& s,
                                    WgradPlan& pl, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  long P = s.pixels();
  bool big = s.cin % 128 == 0 && s.cout % 128 == 0;
  int bm = big ? 128 : 64, bn = big ? 128 : 64;
  int tiles = s.taps * (s.cin / bn) * (s.cout / bm);
  long E = (long)s.cout * s.taps * s.cin;
  pl = wgrad_plan<2, 2>(P, tiles, E);
  if (pl.S == 1)   // a single split writes the gradient itself
    for (int k = 0; k < n; ++k) part[k] = dw[k];
  MbWg io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    const int q = k < n ? k : 0;
    io.x[k] = (const bf16_t*)x[q];
    io.dz[k] = (const bf16_t*)dz[q];
    io.part[k] = part[q];
  }
  dim3 grid(n * s.taps * (s.cin / bn) * (s.cout / bm) * pl.S);
  double flops = 2.0 * n * P * E;
  double bytes = n * (2.0 * ((double)P * s.cin + (double)P * s.cout) + 4.0 * pl.S * E);
  const char* nm = big ? (s.taps == 9 ? "conv_wgrad_mfma<2,2,2,2,9>" : "conv_wgrad_mfma<2,2,2,2,1>")
                       : (s.taps == 9 ? "conv_wgrad_mfma<2,2,1,1,9>" : "conv_wgrad_mfma<2,2,1,1,1>");
  ProfScope ps(nm, flops, bytes, st);
  if (big) {
    if (s.taps == 9)
      TGP_LAUNCH(ps, (conv_wgrad_mfma<2, 2, 2, 2, 9>), grid, dim3(256), 0, st, io, n, (int)P, s.H,
                 s.W, s.cin, s.cout, pl.pix_per_split);
    else
      TGP_LAUNCH(ps, (conv_wgrad_mfma<2, 2, 2, 2, 1>), grid, dim3(256), 0, st, io, n, (int)P, s.H,
                 s.W, s.cin, s.cout, pl.pix_per_split);
  } else {
    if (s.taps == 9)
      TGP_LAUNCH(ps, (conv_wgrad_mfma<2, 2, 1, 1, 9>), grid, dim3(256), 0, st, io, n, (int)P, s.H,
                 s.W, s.cin, s.cout, pl.pix_per_split);
    else
      TGP_LAUNCH(ps, (conv_wgrad_mfma<2, 2, 1, 1, 1>), grid, dim3(256), 0, st, io, n, (int)P, s.H,
                 s.W, s.cin, s.cout, pl.pix_per_split);
  }
  return launch_status();
}

hipError_t conv_wgrad_mfma(const void* x, const void* dz, float* dw, float* partial,
                           const ConvShape& s, hipStream_t st, ReduceJob* defer) {
  if (use_wgrad_rows(s)) return conv_wgrad_rows_launch(x, dz, dw, partial, s, st, defer);
  long E = (long)s.cout * s.taps * s.cin;
  if (use_wgrad_tile(s) || wgrad1x1_tile_ok(s)) {
    return s.taps == 1 ? wgrad1x1_tile_launch(1, &x, &dz, &dw, &partial, s, st, &defer)
                       : conv_wgrad_tile_launch(1, &x, &dz, &dw, &partial, s, st, &defer);
  }
  WgradPlan pl;
  hipError_t e = launch_wgrad_mfma(1, &x, &dz, &dw, &partial, s, pl, st);
  if (e == hipSuccess) *defer = ReduceJob{partial, dw, E, pl.S};   // partial == dw when S == 1
  return e;
}

hipError_t splitk_reduce_n(int n, const float* const* part, float* const* out, long E, int S,
                           hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  SumGroup io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.part[k] = part[k < n ? k : 0];
    io.out[k] = out[k < n ? k : 0];
  }
  int lc = 0;
  while (lc < 6 && (1L << lc) < E) ++lc;
  ProfScope ps("splitk_reduce", 0.0, 4.0 * n * E * (S + 1), st);
  TGP_LAUNCH(ps, splitk_reduce_scalar, dim3(cdiv(E, 1L << lc), n), dim3(256), 0, st, io, E, S, lc);
  return launch_status();
}

hipError_t splitk_reduce_launch(const float* part, float* out, long E, int S, hipStream_t st,
                               const ReduceJob* extra) {
  if (extra && (E % 4 || extra->E % 4)) {   // scalar sums run on their own
    const hipError_t e = splitk_reduce_launch(extra->part, extra->out, extra->E, extra->S, st);
    if (e != hipSuccess) return e;
    extra = nullptr;
  }
  if (E % 4) return splitk_reduce_n(1, &part, &out, E, S, st);
  ProfScope ps("splitk_reduce", 0.0,
               4.0 * E * (S + 1) + (extra ? 4.0 * extra->E * (extra->S + 1) : 0.0), st);
  // many splits of few columns: 16 columns x 64 split lanes; few splits:
  // 256 columns x 4 lanes (chosen by the first sum's S; the second, if any,
  // uses the same layout)
  const int C4 = S >= 64 ? 16 : (S >= 16 ? 64 : 256);
  const int nb1 = (int)cdiv(E, 4L * C4);
  const int nb2 = extra ? (int)cdiv(extra->E, 4L * C4) : 0;
  const float* p2 = extra ? extra->part : nullptr;
  float* o2 = extra ? extra->out : nullptr;
  const long E2 = extra ? extra->E : 0;
  const int S2 = extra ? extra->S : 0;
  if (C4 == 16)
    TGP_LAUNCH(ps, splitk_reduce<16>, dim3(nb1 + nb2), dim3(1024), 0, st, part, out, E, S, p2, o2,
               E2, S2, nb1);
  else if (C4 == 64)
    TGP_LAUNCH(ps, splitk_reduce<64>, dim3(nb1 + nb2), dim3(1024), 0, st, part, out, E, S, p2, o2,
               E2, S2, nb1);
  else
    TGP_LAUNCH(ps, splitk_reduce<256>, dim3(nb1 + nb2), dim3(1024), 0, st, part, out, E, S, p2,
               o2, E2, S2, nb1);
  return launch_status();
}

// Two micro-batches of one layer where the planned kernel takes two tensors
// (the per-tap kernel), else one launch each; the same values as two
// conv_forward_mfma calls either way.
static hipError_t conv_forward_mfma_pair(const void* x0, const void* x1, const void* w,
                                         const float* b, void* y0, void* y1, const ConvShape& s,
                                         int relu, float* part0, float* part1, size_t part_cap,
                                         hipStream_t st) {
  const FwdPlan pl = fwd_plan(s);
  if (pl.cfg >= 100 && pl.cfg < 200) {
    // the per-tap kernel: both micro-batches' tiles in one grid
    const long P = s.pixels();
    const bf16_t* X = (const bf16_t*)x0;
    const bf16_t* X2 = (const bf16_t*)x1;
    const bf16_t* Wt = (const bf16_t*)w;
    bf16_t* Y = (bf16_t*)y0;
    bf16_t* Y2 = (bf16_t*)y1;
    switch (pl.cfg - 100) {
      case 1: return TGP_FWD_CFG(2, 2, 1, 1, 2);
      case 2: return TGP_FWD_CFG(2, 4, 1, 1, 2);
      default: return P >= 32768 && s.cout <= 128 ? TGP_FWD_CFG(2, 4, 1, 1, 2)
                                                   : TGP_FWD_CFG(2, 2, 1, 1, 2);
    }
  }
  hipError_t e = conv_forward_mfma(x0, w, b, y0, s, relu, part0, part_cap, st);
  if (e != hipSuccess) return e;
  return conv_forward_mfma(x1, w, b, y1, s, relu, part1, part_cap, st);
}

// n micro-batches of one layer: one launch of the nine-tap or resident-
// weight 1x1 kernel where it is planned, else pairs (and a single for odd n).
hipError_t conv_forward_mfma_n(int n, const void* const* x, const void* w, const float* b,
                               void* const* y, const ConvShape& s, int relu, float* const* part,
                               size_t part_cap, hipStream_t st) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  const FwdPlan pl = fwd_plan(s);
  if (tile_instead(pl, s, n))
    return launch_tile_cfg(FwdPlan{500, 1}, n, x, w, b, y, s, relu, false, nullptr, 0, st);
  if (pl.cfg == 150) return launch_1x1_res(n, x, (const bf16_t*)w, b, y, s, relu, st);
  if (pl.cfg >= 500)
    return launch_tile_cfg(pl, n, x, w, b, y, s, relu, false, part, part_cap, st);
  if (pl.cfg >= 400) {
    g_rows32_cfg = pl.cfg >= 401 ? pl.cfg - 401 : -1;
    const hipError_t e = conv_forward_rows32(n, x, w, b, y, s, relu, st);
    g_rows32_cfg = -1;
    return e;
  }
  for (int k = 0; k < n; k += 2) {
    const hipError_t e =
        k + 1 < n ? conv_forward_mfma_pair(x[k], x[k + 1], w, b, y[k], y[k + 1], s, relu, part[k],
                                           part[k + 1], part_cap, st)
                  : conv_forward_mfma(x[k], w, b, y[k], s, relu, part[k], part_cap, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The weight gradients of n micro-batches in one launch, every sum left
// pending: the row-blocked kernel where it applies, else the per-tap one.
hipError_t conv_wgrad_mfma_n(int n, const void* const* x, const void* const* dz,
                             float* const* dw, float* const* part, const ConvShape& s,
                             hipStream_t st, ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  if (use_wgrad_rows(s)) return conv_wgrad_rows_launch_n(n, x, dz, dw, part, s, st, defer);
  if (use_wgrad_tile(s)) return conv_wgrad_tile_launch(n, x, dz, dw, part, s, st, defer);
  if (wgrad1x1_tile_ok(s)) return wgrad1x1_tile_launch(n, x, dz, dw, part, s, st, defer);
  const long E = (long)s.cout * s.taps * s.cin;
  WgradPlan pl;
  float* pp[kMaxGroup];
  for (int k = 0; k < n; ++k) pp[k] = part[k];
  hipError_t e = launch_wgrad_mfma(n, x, dz, dw, pp, s, pl, st);
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{pp[k], dw[k], E, pl.S};   // pp == dw when S == 1
  return hipSuccess;
}

}  // namespace tgpk
