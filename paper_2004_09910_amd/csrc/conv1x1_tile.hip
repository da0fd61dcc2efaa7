// bf16 1x1 convolution (forward and data gradient) and its weight gradient
// for any channel counts that are multiples of 8, on 32 x 32 x 16 MFMA.
//
// Forward: Y^T[co][p] = sum_ci W[co][ci] X[p][ci], a GEMM whose both operands
// are contiguous in the sum.  A block's tile is BN channels x BM pixels; a
// stage holds 64 channels of both (128-byte LDS rows, 16-byte chunks
// XOR-swizzled).  The data gradient (DG) reads the forward weights as rows of
// BN channels per sum channel and gathers fragments with the transpose loads,
// so no transposed copy is made.  Weight gradient: dW[co][ci] = sum_p dZ[p][co]
// X[p][ci], both operands pixel-major rows gathered by the transpose loads.
// Channels past the counts and pixels past the end are buffer reads at
// out-of-range offsets (zeros); stores leave them out.
//
// These layers read and write about as long as they multiply, so what bounds
// them is memory and, for small ones, the launch: blocks are persistent over
// tiles (K ranges) with the next one's stages in flight, and a launch takes a
// whole group of micro-batches.  Measured against the per-tap kernels (two
// micro-batches a launch, weights transposed first), us: 256 -> 1024 at 28 x
// 28 x 4, two micro-batches, forward 13.5 -> 12.1, data gradient 13.5 + 4 ->
// 11.8, weight gradient 15.6 -> 12.8; 128 -> 512 at 112 x 112 x 4, two, 62 ->
// 49, 31 -> 28, 47 -> 42; 192 -> 192 at 28 x 28 x 3, four, 18 -> 5.4, 18 ->
// 5.0, 10.1 -> 9.7.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {



struct Io1x1 {
  const bf16_t* x[kMaxGroup];
  bf16_t* y[kMaxGroup];
};

// WC x WP waves, a wave's tile 32 MT channels x 32 FW pixels.
template <int MT, int WC, int WP, int FW, int NS, bool DG>
__global__ __launch_bounds__(WC * WP * 64) void conv1x1_tile(Io1x1 io, int ng,
                                                             const bf16_t* __restrict__ Wt,
                                                             const float* __restrict__ bias, int P,
                                                             int Cin, int Cout, int relu) {
  constexpr int NW = WC * WP, BN = 32 * MT * WC, BM = 32 * WP * FW;
  constexpr int ACH = BN / 8;                                   // weight chunks (1 KiB) per stage
  constexpr int CH = ACH + BM / 8;                              // chunks per stage
  constexpr int LW = CH / NW;                                   // ... per wave
  constexpr int SB = CH * 1024;
  constexpr int RAB = 2 * BN, RPC = 1024 / RAB;                 // (DG) bytes of a weight row, rows per chunk
  static_assert(CH % NW == 0 && ACH % NW == 0, "whole DMA rounds");
  static_assert(NS * SB <= 160 * 1024, "LDS ring");
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * SB];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave % WP, wc = wave / WP;
  const int nct = (Cout + BN - 1) / BN, npt = (P + BM - 1) / BM;
  const int items = ng * npt * nct;
  const int G = gridDim.x;
  const int lb = xcd_remap(blockIdx.x, G);
  const int n_items = lb < items ? (items - lb + G - 1) / G : 0;
  const int nk = (Cin + 63) / 64;
  const int total = n_items * nk;
  const u32x4 rw = make_rsrc(Wt, Cout * Cin * 2);

  // DMA: instruction u of this wave fills chunk NW u + wave; the first ACH
  // chunks are weights (8 channels' rows of 64 sum channels, or (DG) RPC sum
  // channels' rows of BN), the rest 8 pixels' rows of 64 channels.
  const int r8 = lane >> 3;
  int aoff[ACH / NW], ak[ACH / NW], ac[ACH / NW], prow[LW - ACH / NW], pc[LW - ACH / NW];
  auto wswz = [](int row) __attribute__((always_inline)) { return BN >= 64 ? 2 * (row & 3) : 0; };
#pragma unroll
  for (int u = 0; u < ACH / NW; ++u) {
    const int k = NW * u + wave;
    if constexpr (DG) {
      const int kk = k * RPC + lane / (64 / RPC);               // sum channel of the stage
      const int c = (lane % (64 / RPC)) ^ wswz(kk);
      aoff[u] = (kk * Cout + 8 * c) * 2;
      ak[u] = kk;
      ac[u] = 8 * c;
    } else {
      const int row = k * 8 + r8, c = swz(row, lane & 7);
      aoff[u] = (row * Cin + 8 * c) * 2;
      ak[u] = 8 * c;
      ac[u] = row;
    }
  }
#pragma unroll
  for (int u = 0; u < LW - ACH / NW; ++u) {
    prow[u] = (NW * u + wave) * 8 + r8;
    pc[u] = 8 * swz(prow[u], lane & 7);
  }

  auto coords = [&](int it, int& gi, int& p0, int& co0) __attribute__((always_inline)) {
    const int item = lb + it * G;
    const int rest = item / nct;
    co0 = (item - rest * nct) * BN;
    gi = rest / npt;
    p0 = (rest - gi * npt) * BM;
  };
  int i_it = 0, i_ks = 0, i_gi = 0, i_p0 = 0, i_co0 = 0;
  if (total > 0) coords(0, i_gi, i_p0, i_co0);
  u32x4 rx = make_rsrc(pickg(io.x, i_gi), P * Cin * 2);
  auto issue = [&](int slot) __attribute__((always_inline)) {
    const int c0 = i_ks * 64;
    const int wo = DG ? (c0 * Cout + i_co0) * 2 : (i_co0 * Cin + c0) * 2;
#pragma unroll
    for (int u = 0; u < ACH / NW; ++u) {
      const bool ok = c0 + ak[u] < Cin && i_co0 + ac[u] < Cout;
      dma16(rw, TGP_LDS(ring + slot * SB + (NW * u + wave) * 1024), ok ? aoff[u] + wo : kOob, 0);
    }
#pragma unroll
    for (int u = 0; u < LW - ACH / NW; ++u) {
      const int p = i_p0 + prow[u];
      const bool ok = p < P && c0 + pc[u] < Cin;
      dma16(rx, TGP_LDS(ring + slot * SB + (ACH + NW * u + wave) * 1024),
            ok ? (p * Cin + c0 + pc[u]) * 2 : kOob, 0);
    }
    if (++i_ks == nk) {
      i_ks = 0;
      if (++i_it < n_items) {
        coords(i_it, i_gi, i_p0, i_co0);
        rx = make_rsrc(pickg(io.x, i_gi), P * Cin * 2);
      }
    }
  };
#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < total) issue(k);

  const int kb = 8 * (lane >> 5) + ((lane & 15) >> 2);          // (DG) row of the transpose load
  int idx = 0;
  for (int it = 0; it < n_items; ++it) {
    int gi, p0, co0;
    coords(it, gi, p0, co0);
    // this lane's bias values, loaded up front (channels co0 + 32 (MT wc + i) +
    // 8 g + 4 (l / 32) + t)
    f32x4_t bv[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int co = co0 + (MT * wc + i) * 32 + 8 * g + 4 * (lane >> 5);
        bv[i][g] = bias && co < Cout ? *(const f32x4_t*)(bias + co) : f32x4_t{};
      }
    f32x16_t acc[MT][FW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < FW; ++j) acc[i][j] = f32x16_t{};
    for (int ks = 0; ks < nk; ++ks, ++idx) {
      wait_stages<NS, LW>(min(NS - 2, total - 1 - idx));
      ring_barrier();
      if (idx + NS - 1 < total) issue((idx + NS - 1) % NS);
      const unsigned char* As = ring + (idx % NS) * SB;
      const unsigned char* Bs = As + ACH * 1024;
      const int left = Cin - ks * 64;                           // (uniform) channels left
      bf16x8_t a[2][MT], b[2][FW];
      auto load = [&](int kk, int buf) __attribute__((always_inline)) {
        const int qq = 2 * kk + (lane >> 5);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          if constexpr (DG) {
            const int cb = ((wc * MT + i) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
            a[buf][i] = as_bf16x8(frag_tr(As + (16 * kk + kb) * RAB + (((cb >> 4) ^ wswz(kb)) << 4) + (cb & 15), RAB));
          } else {
            const int row = (wc * MT + i) * 32 + (lane & 31);
            a[buf][i] = as_bf16x8(*(const u32x4*)(As + row * 128 + swz(row, qq) * 16));
          }
        }
#pragma unroll
        for (int j = 0; j < FW; ++j) {
          const int row = (wp * FW + j) * 32 + (lane & 31);
          b[buf][j] = as_bf16x8(*(const u32x4*)(Bs + row * 128 + swz(row, qq) * 16));
        }
      };
      // the fragments of K sub-step kk + 1 are read while the MFMAs of kk run;
      // sub-steps past the last channel are left out
      load(0, 0);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        if (16 * kk >= left) break;
        if (kk + 1 < 4) load(kk + 1, (kk + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < FW; ++j) acc[i][j] = mfma32(a[kk & 1][i], b[kk & 1][j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Epilogue: lanes l and l + 32 hold channels 8 g + 0..3 and 8 g + 4..7 of
    // pixel l % 32; swapping the halves of groups 2 h and 2 h + 1 across the
    // half-waves leaves each lane 8 consecutive channels, one 16-byte store.
    bf16_t* __restrict__ Y = pickg(io.y, gi);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
#pragma unroll
      for (int j = 0; j < FW; ++j) {
        const int p = p0 + (wp * FW + j) * 32 + (lane & 31);
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
          const int co = co0 + (wc * MT + i) * 32 + 16 * h + 8 * (lane >> 5);
          if (p < P && co < Cout)
            *(u32x4*)(Y + (long)p * Cout + co) =
                u32x4{pk[2 * h][0], pk[2 * h][1], pk[2 * h + 1][0], pk[2 * h + 1][1]};
        }
      }
    }
  }
}

// ---------------------------------------------------------------- weight gradient

struct Wg1x1 {
  const bf16_t* x[kMaxGroup];
  const bf16_t* dz[kMaxGroup];
  float* out[kMaxGroup];
};

// An item is (K range, 64 MC output channels, 64 NC input channels); 2 x 2
// waves, a wave's tile 32 MC x 32 NC.  A stage is 64 pixels: MC planes of dZ
// rows and NC planes of input rows, 64 channels (128 bytes) a row, 16-byte
// chunks swizzled by 2 (row & 3).
template <int MC, int NC, int NS>
__global__ __launch_bounds__(256) void wgrad1x1_tile(Wg1x1 io, int ng, int P, int Cin, int Cout,
                                                     int nK, int spk) {
  constexpr int NPL = MC + NC, SB = NPL * 8192, LW = 2 * NPL;
  static_assert(NS * SB <= 160 * 1024, "LDS ring");
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * SB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int ncit = (Cin + 64 * NC - 1) / (64 * NC), nct = (Cout + 64 * MC - 1) / (64 * MC);
  const int per_k = nct * ncit;
  const int items = ng * nK * per_k;
  const int G = gridDim.x;
  const int lb = xcd_remap(blockIdx.x, G);
  const int n_items = lb < items ? (items - lb + G - 1) / G : 0;
  const int T = (P + 63) / 64;
  const long E = (long)Cout * Cin;

  auto coords = [&](int it, int& kr, int& co0, int& ci0, int& s0) __attribute__((always_inline)) {
    const int item = lb + it * G;
    kr = item / per_k;
    const int t = item - kr * per_k;
    co0 = (t / ncit) * 64 * MC;
    ci0 = (t % ncit) * 64 * NC;
    s0 = (kr % nK) * spk;
    return min(spk, T - s0);                                    // stages
  };
  int total = 0;
  for (int it = 0; it < n_items; ++it) {
    int kr, co0, ci0, s0;
    total += coords(it, kr, co0, ci0, s0);
  }
  // DMA: instruction u of this wave fills chunk 4 u + wave: plane chunk / 8,
  // rows 8 (chunk % 8) + lane / 8
  int i_it = 0, i_st = 0, i_n = 0, i_s0 = 0, i_co0 = 0, i_ci0 = 0;
  u32x4 rz = {}, rx = {};
  auto item_on = [&]() __attribute__((always_inline)) {
    int kr;
    i_n = coords(i_it, kr, i_co0, i_ci0, i_s0);
    rz = make_rsrc(pickg(io.dz, kr / nK), P * Cout * 2);
    rx = make_rsrc(pickg(io.x, kr / nK), P * Cin * 2);
  };
  if (n_items > 0) item_on();
  const int rl = lane >> 3, lc = (lane & 7) ^ (2 * (rl & 3));
  auto issue = [&](int slot) __attribute__((always_inline)) {
    const int pb = (i_s0 + i_st) * 64;
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int c = 4 * u + wave, pl = c >> 3;                  // plane: u / 2
      const int p = pb + 8 * (c & 7) + rl;
      auto* dst = TGP_LDS(ring + slot * SB + c * 1024);
      if (pl < MC) {
        const int ch = i_co0 + 64 * pl + 8 * lc;
        dma16(rz, dst, p < P && ch < Cout ? (p * Cout + ch) * 2 : kOob, 0);
      } else {
        const int ch = i_ci0 + 64 * (pl - MC) + 8 * lc;
        dma16(rx, dst, p < P && ch < Cin ? (p * Cin + ch) * 2 : kOob, 0);
      }
    }
    if (++i_st == i_n) {
      i_st = 0;
      if (++i_it < n_items) item_on();
    }
  };
#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < total) issue(k);

  // Fragment constants: lane group g = lane / 16 holds channels 16 (g % 2) ..
  // + 15 and pixels 8 (g / 2) .. + 7; lane j of it addresses pixel j / 4,
  // channels 4 (j % 4) .. + 3.  Wave channel tile q (32 channels) lies in plane
  // q / 2, half q % 2.
  const int kb = 8 * (lane >> 5) + ((lane & 15) >> 2);
  auto fbase = [&](int q) __attribute__((always_inline)) {
    const int cb = ((q & 1) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
    return (q >> 1) * 8192 + kb * 128 + (((cb >> 4) ^ (2 * (kb & 3))) << 4) + (cb & 15);
  };
  int fa[MC], fb[NC];
#pragma unroll
  for (int i = 0; i < MC; ++i) fa[i] = fbase(wm * MC + i);
#pragma unroll
  for (int j = 0; j < NC; ++j) fb[j] = MC * 8192 + fbase(wn * NC + j);

  int idx = 0;
  for (int it = 0; it < n_items; ++it) {
    int kr, co0, ci0, s0;
    const int ns = coords(it, kr, co0, ci0, s0);
    f32x16_t acc[MC][NC];
#pragma unroll
    for (int i = 0; i < MC; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j) acc[i][j] = f32x16_t{};
    for (int st = 0; st < ns; ++st, ++idx) {
      wait_stages<NS, LW>(min(NS - 2, total - 1 - idx));
      ring_barrier();
      if (idx + NS - 1 < total) issue((idx + NS - 1) % NS);
      const unsigned char* sp = ring + (idx % NS) * SB;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8_t a[MC], b[NC];
#pragma unroll
        for (int i = 0; i < MC; ++i) a[i] = as_bf16x8(frag_tr(sp + fa[i] + kk * 16 * 128, 128));
#pragma unroll
        for (int j = 0; j < NC; ++j) b[j] = as_bf16x8(frag_tr(sp + fb[j] + kk * 16 * 128, 128));
#pragma unroll
        for (int i = 0; i < MC; ++i)
#pragma unroll
          for (int j = 0; j < NC; ++j) acc[i][j] = mfma32(a[i], b[j], acc[i][j]);
      }
    }
    const int gi = kr / nK;
    float* o = pickg(io.out, gi) + (long)(kr - gi * nK) * E;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int ci = ci0 + (wn * NC + j) * 32 + (lane & 31);
      if (ci >= Cin) continue;
#pragma unroll
      for (int i = 0; i < MC; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int co = co0 + (wm * MC + i) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          if (co < Cout) o[(long)co * Cin + ci] = acc[i][j][v];
        }
    }
  }
}

// ---------------------------------------------------------------- rules

struct Cfg1x1 { int MT, WC, WP, FW, NS; };
constexpr Cfg1x1 kCfg1x1[] = {
    {2, 2, 4, 1, 2},   // 128 channels x 128 pixels, eight waves
    {1, 2, 4, 1, 2},   // 64 x 128, eight waves
    {1, 2, 2, 1, 3},   // 64 x 64, four waves
    {1, 1, 4, 1, 2},   // 32 x 128, four waves
    {1, 2, 2, 1, 6},   // 64 x 64, four waves, deep ring
};

}  // namespace

thread_local int g_1x1_cfg = -1;   // >= 0 forces a configuration (tests and measurement)

// Tile for ng micro-batches: the largest whose tiles fill a round of blocks;
// where 64 x 64 tiles do not, a deep ring, since a block's few loads in flight
// then set the time.  (us: 512 -> 512, 25088 pixels: 29 with 128 x 128, 30 with
// 64 x 128, 35 with 64 x 64; 64-channel outputs, 100352 pixels: 17.5, 11.9,
// 12.9.  The per-tap kernel, two micro-batches a launch: 78 and 17.)
static int pick1x1(const ConvShape& s, int ng) {
  if (g_1x1_cfg >= 0) return g_1x1_cfg;
  if (s.cout <= 32) return 3;
  const long P = ng * s.pixels();
  if (s.cout > 64 && (P / 128) * ((s.cout + 127) / 128) >= 256) return 0;
  const long c64 = (s.cout + 63) / 64;
  if ((P / 128) * c64 >= 256) return 1;
  return s.cin > 192 && (P + 63) / 64 * c64 <= 256 ? 4 : 2;
}

bool conv1x1_tile_ok(const ConvShape& s) {
  return s.taps == 1 && s.cin % 8 == 0 && s.cout % 8 == 0 && s.pixels() > 0 &&
         (double)s.pixels() * s.cin * 2 < 2147483648.0 - 65536 &&
         (double)s.cout * s.cin * 2 < 2147483648.0 - 65536;
}

template <int MT, int WC, int WP, int FW, int NS, bool DG>
static hipError_t launch1x1(const Io1x1& io, int ng, const bf16_t* Wt, const float* b,
                            const ConvShape& s, int relu, hipStream_t st) {
  static const KernelName name("conv1x1_tile<%d,%d,%d,%d%s>", MT, WC, WP, FW, DG ? ",dg" : "");
  constexpr int BN = 32 * MT * WC, BM = 32 * WP * FW, LDS = NS * (BN + BM) * 128;
  const long P = s.pixels();
  const long items = (long)ng * ((P + BM - 1) / BM) * ((s.cout + BN - 1) / BN);
  if (items >= (1L << 31)) return hipErrorInvalidValue;
  constexpr int occ = LDS * 5 <= 160 * 1024 ? 5 : LDS * 3 <= 160 * 1024 ? 3 : LDS * 2 <= 160 * 1024 ? 2 : 1;
  const int G = (int)(items < 256 * occ ? items : 256 * occ);
  ProfScope ps(name.s, 2.0 * ng * P * s.cout * s.cin,
               2.0 * ((double)ng * P * (s.cin + s.cout) + (double)s.cout * s.cin), st);
  TGP_LAUNCH(ps, (conv1x1_tile<MT, WC, WP, FW, NS, DG>), dim3(G), dim3(WC * WP * 64), 0, st, io, ng,
             Wt, b, (int)P, s.cin, s.cout, relu);
  return launch_status();
}

hipError_t conv_forward_1x1(int n, const void* const* x, const void* w, const float* b,
                            void* const* y, const ConvShape& s, int relu, bool dg,
                            hipStream_t st) {
  if (n < 1 || n > kMaxGroup || !conv1x1_tile_ok(s) || !w) return hipErrorInvalidValue;
  Io1x1 io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.y[k] = (bf16_t*)y[k < n ? k : 0];
  }
  const bf16_t* Wt = (const bf16_t*)w;
  switch (pick1x1(s, n)) {
#define C1_GO(i, D)                                                                           \
  launch1x1<kCfg1x1[i].MT, kCfg1x1[i].WC, kCfg1x1[i].WP, kCfg1x1[i].FW, kCfg1x1[i].NS, D>(    \
      io, n, Wt, b, s, relu, st)
#define C1_CASE(i) \
  case i: return dg ? C1_GO(i, true) : C1_GO(i, false);
    C1_CASE(0) C1_CASE(1) C1_CASE(2) C1_CASE(3) C1_CASE(4)
#undef C1_CASE
#undef C1_GO
    default: return hipErrorInvalidValue;
  }
}

// K ranges of one micro-batch: twelve stages of 64 pixels each, since a range's
// sums are written and read once more (256 x 256, 12544 pixels, sixteen
// micro-batches: 32 ranges 68 us, 16 58), but at least 128 items of 64 x 64 and
// at most 512; at most 8 MB of slices and no more than the general kernels'.
struct Plan1x1 { int nK, spk; };
static Plan1x1 wg1x1_plan(const ConvShape& s) {
  const long t64 = (long)((s.cout + 63) / 64) * ((s.cin + 63) / 64);
  const long T = (s.pixels() + 63) / 64, E = (long)s.cout * s.cin;
  const long want = std::min((512 + t64 - 1) / t64, std::max(T / 12, (128 + t64 - 1) / t64));
  const long nK = std::max(1L, std::min({T, want, std::max(1L, (8L << 20) / (4 * E)),
                                         (long)wgrad_general_splits(s)}));
  const int spk = (int)((T + nK - 1) / nK);
  return {(int)((T + spk - 1) / spk), spk};
}

bool wgrad1x1_tile_ok(const ConvShape& s) {
  return conv1x1_tile_ok(s) && (double)s.pixels() * s.cout * 2 < 2147483648.0 - 65536;
}
size_t wgrad1x1_tile_partial_floats(const ConvShape& s) {
  const Plan1x1 p = wg1x1_plan(s);
  return p.nK > 1 ? (size_t)p.nK * s.cout * s.cin : 0;
}

hipError_t wgrad1x1_tile_launch(int n, const void* const* x, const void* const* dz,
                                float* const* dw, float* const* partial, const ConvShape& s,
                                hipStream_t st, ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup || !wgrad1x1_tile_ok(s)) return hipErrorInvalidValue;
  const Plan1x1 p = wg1x1_plan(s);
  Wg1x1 io;
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    const int q = k < n ? k : 0;
    io.x[k] = (const bf16_t*)x[q];
    io.dz[k] = (const bf16_t*)dz[q];
    io.out[k] = p.nK > 1 ? partial[q] : dw[q];
  }
  const long E = (long)s.cout * s.cin;
  // 128 x 128 items where they give every CU one (the sums of an element run
  // over the same pixels in the same order either way)
  const long big = (long)n * p.nK * ((s.cout + 127) / 128) * ((s.cin + 127) / 128);
  const int MC = s.cin > 64 && s.cout > 64 && big >= 256 ? 2 : 1;
  const long items = MC == 2 ? big : (long)n * p.nK * ((s.cout + 63) / 64) * ((s.cin + 63) / 64);
  {
    ProfScope ps(MC == 2 ? "wgrad1x1_tile<2,2>" : "wgrad1x1_tile<1,1>", 2.0 * n * s.pixels() * E,
                 n * (2.0 * s.pixels() * (s.cin + s.cout) + 4.0 * p.nK * E), st);
    if (MC == 2) {
      const int G = (int)(items < 512 ? items : 512);
      TGP_LAUNCH(ps, (wgrad1x1_tile<2, 2, 2>), dim3(G), dim3(256), 0, st, io, n, (int)s.pixels(),
                 s.cin, s.cout, p.nK, p.spk);
    } else {
      const int G = (int)(items < 768 ? items : 768);
      TGP_LAUNCH(ps, (wgrad1x1_tile<1, 1, 3>), dim3(G), dim3(256), 0, st, io, n, (int)s.pixels(),
                 s.cin, s.cout, p.nK, p.spk);
    }
  }
  const hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{io.out[k], dw[k], E, p.nK};
  return hipSuccess;
}

}  // namespace tgpk
