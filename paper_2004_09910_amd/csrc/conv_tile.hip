// bf16 3x3 convolution (forward and data gradient) for any image size and any
// channel counts that are multiples of 8, on 32 x 32 x 16 MFMA with
// rectangular pixel tiles and all nine taps per stage.
//
// An output tile is BN output channels x (R rows x TW columns) of one sample.
// R and TW are launch arguments: an image is cut into equal column strips and
// row blocks so that a tile fills the kernel's pixel fragments as well as the
// image allows.  The K loop runs over 16-channel chunks of the input; a stage
// holds in LDS, for one chunk, the weights of all nine taps for the BN
// channels (tap-major) and the R + 2 input rows of the tile, each as a block
// of BWP LDS rows (TW + 2 rounded up to a multiple of 16, the first and last
// pixel being the halo).  Every LDS row is 16 channels (32 bytes), its
// 16-byte halves swapped when bit 3 of the row index is set: a fragment of 32
// consecutive rows is then read without bank conflicts from any start row,
// and a filter-row shift is a constant offset.  Pixels outside the image,
// channels past Cin and output channels past Cout are buffer reads at
// out-of-range offsets and hold zeros; the stores leave them out.
//
// The data gradient (DG) is the same sum with the filter rotated and its
// channels exchanged.  It reads the forward weights as they are: a stage's
// weights are then rows of BN channels for each (tap, sum channel), and the
// transpose loads gather a fragment's sum channels from them.  So no
// transposed copy of the weights is made or kept (64 -> 64 channels at 56 x
// 56, one sample: one launch of 4 us less of a step of 32).
//
// What bounds it: per tap a wave reads MT + FW fragments of 1 KiB for MT FW MFMAs,
// so wide layers take MT = FW = 2 (128 channels x 256 pixels a block) or FW = 4 (64 x
// 512); few tiles or few channels take the smaller tiles.  At 128 channels, 56 x
// 56 x 8, four micro-batches (64 x 512 tiles) the MFMAs are busy 31% of the time, LDS
// 30%, and waves wait a third of theirs: one block a CU, whose stages hand over
// behind a barrier.  The sum of an output runs over (chunk, tap, channel) in every configuration, so the
// choice does not change values and a recomputation is bit-identical.
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {


typedef __bf16 bf16x2_ct __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack2_ct(float a, float b) {
  const bf16x2_ct h = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(unsigned, h);
}

// The micro-batches of one launch (nb samples each, the same weights); their
// tiles share the persistent grid.  A larger group runs as launches of eight.
constexpr int kTileGroup = 8;
struct TileIo {
  const bf16_t* x[kTileGroup];
  bf16_t* y[kTileGroup];
  float* part[kTileGroup];   // split K: S sums of every output
};
// How an image is cut: R rows x TW columns a tile, BWP LDS rows per input
// row, nrb row blocks and ns column strips; inv = ceil(2^20 / TW), invB =
// ceil(2^20 / BWP) (exact quotients for a tile's pixels and a slot's rows).  TALL:
// hp is H + 1 and invH = ceil(2^20 / hp) (exact for kTallRows rows and a tile more).
struct TileCut {
  int R, TW, BWP, nrb, ns, inv, invB, hp, invH;
};
constexpr int kTallRows = 1024;

// WC x WP waves; a wave covers MT 32-channel tiles x FW pixel fragments.  LW
// is the DMA instructions of a wave per stage (1 KiB each), which fixes the
// slot size; chunks past the stage's rows read zeros.
// With SPLIT an item is a tile's share of the sum, 1 / S of its stages, whose
// float32 sums go to part; the items of one share of one channel tile are
// neighbours, so that an XCD reads its weights once.
// With TALL a tile spans samples: a micro-batch is one image of nb (H + 1) - 1 rows,
// the row after each sample a zero row that is the halo of both its neighbours and
// whose outputs are left out.
template <int MT, int WC, int WP, int FW, int LW, int NS, bool DG, bool SPLIT, bool TALL>
__global__ __launch_bounds__(WC * WP * 64) void conv3x3_tile(
    TileIo io, int ng, const bf16_t* __restrict__ Wt, const float* __restrict__ bias, int nb,
    int H, int W, int Cin, int Cout, int relu, int S, TileCut cut) {
  constexpr int NW = WC * WP;
  constexpr int NQ = MT * FW;                                   // MFMAs per tap
  constexpr int BN = 32 * MT * WC;
  constexpr int AR = 9 * BN;                                    // weight rows per stage
  constexpr int ACH = AR / 32;                                  // ... in 1 KiB chunks
  constexpr int SB = LW * NW * 1024;                            // slot bytes
  static_assert(NS * SB + (NS + 1) * 1024 <= 160 * 1024, "LDS ring and bias slots");
  static_assert(NW * 2048 * MT <= SB, "epilogue staging fits a slot");
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * SB + (NS + 1) * 1024];
  unsigned char* const bslots = ring + NS * SB;                 // BN bias values per tile in flight

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pg = wave % WP, wc = wave / WP;                     // pixel group, channel group
  const int R = cut.R, TW = cut.TW, BWP = cut.BWP;
  const int nct = (Cout + BN - 1) / BN;
  const int per_n = cut.nrb * cut.ns * nct;                     // tiles per sample
  const int nbv = TALL ? 1 : nb, Hv = TALL ? nb * cut.hp - 1 : H;   // images and rows cut into tiles
  const int items = ng * nbv * per_n * (SPLIT ? S : 1);
  const int G = gridDim.x;
  const int lb = xcd_remap(blockIdx.x, G);
  const int n_items = lb < items ? (items - lb + G - 1) / G : 0;
  const int nk = (Cin + 15) / 16 / (SPLIT ? S : 1);             // stages per item (S divides)
  const int total = n_items * nk;

  const int xbytes = nb * H * W * Cin * 2;                      // one micro-batch's input
  constexpr int RAB = 2 * BN;                                   // (DG) bytes of a weight row
  constexpr int RPC = 1024 / RAB;                               // ... rows per 1 KiB chunk
  // swizzle of a weight row's 16-byte chunks, for rows of 128 bytes and more
  auto wswz = [](int row) __attribute__((always_inline)) { return BN >= 64 ? 2 * (row & 3) : 0; };
  const u32x4 rw = make_rsrc(Wt, Cout * 9 * Cin * 2);
  const u32x4 rbias = make_rsrc(bias, bias ? Cout * 4 : 0);     // no bias reads zeros

  // DMA: instruction u of this wave fills stage chunk k = NW u + wave; lane l
  // the 16 bytes at + 16 l: row k * 32 + l / 2, physical half l % 2, which
  // holds logical half lh (the same for every chunk of the lane).
  const int lh = (lane & 1) ^ ((lane >> 4) & 1);
  int doff[LW], drc[LW];                                        // byte offset; rr | wp << 16
#pragma unroll
  for (int u = 0; u < LW; ++u) {
    const int k = NW * u + wave;
    const int row = k * 32 + (lane >> 1);
    if (k < ACH && DG) {
      // weight row (tap, sum channel kk) of the rotated filter
      const int wr = k * RPC + lane / (64 / RPC);
      const int tap = wr / 16, kk = wr - 16 * tap;
      const int lc = lane % (64 / RPC) ^ wswz(wr);
      doff[u] = ((kk * 9 + 8 - tap) * Cout + 8 * lc) * 2;
      drc[u] = kk | (lc << 16);
    } else if (k < ACH) {
      const int tap = row / BN, co = row - tap * BN;
      doff[u] = ((co * 9 + tap) * Cin + 8 * lh) * 2;
      drc[u] = 0;
    } else {
      const int q = row - AR;
      const int rr = (q * cut.invB) >> 20, wp = q - rr * BWP;   // q / BWP
      const bool ok = rr < R + 2 && wp < TW + 2;
      doff[u] = ok ? ((rr * W + wp - 1) * Cin + 8 * lh) * 2 : 0;
      drc[u] = ok ? rr | (wp << 16) : -1;
    }
  }

  // Fragment addresses (bytes within a stage).  A: weight row tap BN + 32 (MT
  // wc + i) + l % 32 at logical half l / 32.  B: pixel tp of the tile at
  // column tap s is LDS row rho BWP + w + s of the input region; filter row r
  // adds r BWP rows.
  // (DG: lane group g = lane / 16 holds channels 16 (g % 2) .. + 15 and sum
  // channels 8 (g / 2) .. + 7; lane j of it addresses row j / 4, channels 4 (j
  // % 4) .. + 3 of the block of 16.)
  const int kb = 8 * (lane >> 5) + ((lane & 15) >> 2);
  int abase[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if constexpr (DG) {
      const int cb = ((wc * MT + i) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
      abase[i] = kb * RAB + (((cb >> 4) ^ wswz(kb)) << 4) + (cb & 15);
    } else {
      abase[i] = ((wc * MT + i) * 32 + (lane & 31)) * 32 + (((lane >> 5) ^ ((lane >> 3) & 1)) << 4);
    }
  }
  int bq[FW][3];
#pragma unroll
  for (int j = 0; j < FW; ++j) {
    int tp = (pg * FW + j) * 32 + (lane & 31);
    tp = min(tp, R * TW - 1);                                   // clamped copy past the tile
    const int rho = (tp * cut.inv) >> 20, w = tp - rho * TW;   // tp / TW
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const int q = rho * BWP + w + s;
      bq[j][s] = AR * 32 + q * 32 + (((lane >> 5) ^ ((q >> 3) & 1)) << 4);
    }
  }

  // item -> micro-batch gi, its sample n, first row h0 and column w0, first
  // output channel co0
  // (SPLIT: and its share sk of the sum)
  auto coords = [&](int it, int& gi, int& n, int& h0, int& w0, int& co0, int& sk)
      __attribute__((always_inline)) {
    const int item = lb + it * G;
    int smp, t, ct;
    if constexpr (SPLIT) {
      const int px = cut.nrb * cut.ns, npx = ng * nbv * px;
      const int sc = item / npx;
      sk = sc / nct;
      ct = sc - sk * nct;
      t = item - sc * npx;
      smp = t / px;
      t -= smp * px;
    } else {
      sk = 0;
      smp = item / per_n;
      t = item - smp * per_n;
      ct = t % nct;
      t /= nct;
    }
    const int sx = t % cut.ns;
    gi = smp / nbv;
    n = smp - gi * nbv;
    h0 = (t / cut.ns) * R;
    w0 = sx * TW;
    co0 = ct * BN;
  };

  int i_it = 0, i_ks = 0, i_gi = 0, i_n = 0, i_h0 = 0, i_w0 = 0, i_co0 = 0, i_sk = 0;
  if (total > 0) coords(0, i_gi, i_n, i_h0, i_w0, i_co0, i_sk);
  u32x4 rxg = make_rsrc(pickg(io.x, i_gi), xbytes);            // the issuing item's input
  auto issue_part = [&](int slot, int u0, int u1) __attribute__((always_inline)) {
    const int c0 = (i_sk * nk + i_ks) * 16;
    const int soff_a = DG ? (c0 * 9 * Cout + i_co0) * 2 : (i_co0 * 9 * Cin + c0) * 2;
    const int hb = i_h0 - 1;                                    // input row of block row 0
    const int base_b = (((i_n * H + hb) * W + i_w0) * Cin + c0) * 2;   // negative for hb = -1
    const bool cok = c0 + 8 * lh < Cin;                         // the last chunk may hold 8 channels
    // the tile's bias values, ahead of its first stage (whose wait covers
    // them): a load in the epilogue would wait for the DMA in flight, and
    // held in registers they spill the widest configuration
    if (!SPLIT && u0 == 0 && i_ks == 0 && wave == 0)
      dma16(rbias, TGP_LDS(bslots + (i_it % (NS + 1)) * 1024),
            lane < BN / 4 ? (i_co0 + 4 * lane) * 4 : kOob, 0);
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      if (u < u0 || u >= u1) continue;
      const int k = NW * u + wave;
      auto* dst = TGP_LDS(ring + slot * SB + k * 1024);
      if (k < ACH) {                                            // wave-uniform
        const bool wok = DG ? c0 + (drc[u] & 0xffff) < Cin && i_co0 + 8 * (drc[u] >> 16) < Cout : cok;
        dma16(rw, dst, wok ? doff[u] + soff_a : kOob, 0);
      } else {
        const int rr = drc[u] & 0xffff, col = i_w0 + (drc[u] >> 16) - 1;
        const int hv = hb + rr, nz = TALL ? (hv * cut.invH) >> 20 : 0;   // zero rows above hv
        const bool ok = drc[u] >= 0 && cok && (unsigned)hv < (unsigned)Hv &&
                        (unsigned)col < (unsigned)W && (!TALL || hv - nz * cut.hp < H);
        dma16(rxg, dst, ok ? base_b + doff[u] - nz * W * Cin * 2 : kOob, 0);
      }
    }
  };
  auto issue_done = [&]() __attribute__((always_inline)) {
    if (++i_ks == nk) {
      i_ks = 0;
      if (++i_it < n_items) {
        coords(i_it, i_gi, i_n, i_h0, i_w0, i_co0, i_sk);
        rxg = make_rsrc(pickg(io.x, i_gi), xbytes);
      }
    }
  };

#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < total) {
      issue_part(k, 0, LW);
      issue_done();
    }

  int idx = 0;
  for (int c_it = 0; c_it < n_items; ++c_it) {
    int gi, n, h0, w0, co0, sk;
    coords(c_it, gi, n, h0, w0, co0, sk);
    f32x16_t acc[MT][FW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < FW; ++j) acc[i][j] = f32x16_t{};

    for (int ks = 0; ks < nk; ++ks, ++idx) {
      // loads complete in order: stage idx is in once at most the stages
      // issued after it are pending (epilogue stores only lengthen the wait)
      wait_stages<NS, LW>(min(NS - 2, total - 1 - idx));
      ring_barrier();
      const bool fill = idx + NS - 1 < total;                   // refill the slot freed last stage
      const int fslot = (idx + NS - 1) % NS;
      const unsigned char* st = ring + (idx % NS) * SB;
      // nine taps; tap t + 1's fragments are read while tap t's MFMAs run
      bf16x8_t fa[2][MT], fb[2][FW];
      auto load = [&](int t, int buf) __attribute__((always_inline)) {
        const int r = t / 3, s = t - 3 * (t / 3);
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if constexpr (DG) {
            fa[buf][i] = as_bf16x8(frag_tr(st + abase[i] + t * 16 * RAB, RAB));
          } else {
            fa[buf][i] = as_bf16x8(*(const u32x4*)(st + abase[i] + t * BN * 32));
          }
#pragma unroll
        for (int j = 0; j < FW; ++j)
          fb[buf][j] = as_bf16x8(*(const u32x4*)(st + bq[j][s] + r * BWP * 32));
      };
      load(0, 0);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        // reads for tap t + 1, half of tap t's MFMAs, this tap's share of the
        // next stage's DMA, the other half of the MFMAs
        if (t + 1 < 9) load(t + 1, (t + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (q < (NQ + 1) / 2)
            acc[q % MT][q / MT] = mfma32(fa[t & 1][q % MT], fb[t & 1][q / MT], acc[q % MT][q / MT]);
        __builtin_amdgcn_sched_barrier(0);
        if (fill) issue_part(fslot, t * LW / 9, (t + 1) * LW / 9);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          if (q >= (NQ + 1) / 2)
            acc[q % MT][q / MT] = mfma32(fa[t & 1][q % MT], fb[t & 1][q / MT], acc[q % MT][q / MT]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (fill) issue_done();
    }

    if constexpr (SPLIT) {
      float* const pt = pickg(io.part, gi) + (long)sk * nb * H * W * Cout;
#pragma unroll
      for (int j = 0; j < FW; ++j) {
        const int tp = (pg * FW + j) * 32 + (lane & 31);
        const int rho = (tp * cut.inv) >> 20, w = tp - rho * TW;
        const int hv = h0 + rho, nz = TALL ? (hv * cut.invH) >> 20 : 0;
        if (rho >= R || hv >= Hv || w0 + w >= W || (TALL && hv - nz * cut.hp >= H)) continue;
        float* const row = pt + ((long)(n * H + hv - nz) * W + w0 + w) * Cout;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int co = co0 + (wc * MT + i) * 32 + 8 * g + 4 * (lane >> 5);
            if (co < Cout)
              *(float4*)(row + co) = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1],
                                                 acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
          }
      }
      continue;
    }
    // Epilogue, staged through LDS so that every store writes whole runs of
    // one pixel's channels.  The slot of the stage just consumed is free once
    // every wave is past its last reads; its refill is issued only after the
    // next stage's barrier.  Per fragment each wave uses its own 32 pixel rows
    // of 32 MT channels, 16-byte chunk c of row p at position c ^ (p % NCK).
    // Element v of lane l of acc[i][j] is channel 32 i + 8 (v / 4) + 4 (l /
    // 32) + v % 4 of pixel l % 32.
    ring_barrier();
    constexpr int ROWB = 64 * MT;                               // staged bytes per pixel
    constexpr int NCK = 4 * MT;                                 // 16-byte chunks per pixel
    constexpr int PPI = 64 / NCK;                               // pixels per read
    unsigned char* ep = ring + ((idx - 1) % NS) * SB + wave * 32 * ROWB;
    const unsigned char* bl =
        bslots + (c_it % (NS + 1)) * 1024 + (32 * MT * wc + 4 * (lane >> 5)) * 4;
    bf16_t* const Yg = pickg(io.y, gi);
    const int pw = lane & 31, hw = lane >> 5;
#pragma unroll
    for (int j = 0; j < FW; ++j) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4_t bv = *(const f32x4_t*)(bl + (32 * i + 8 * g) * 4);
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = acc[i][j][4 * g + e] + bv[e];
            if (relu) v[e] = fmaxf(v[e], 0.0f);
          }
          uint2 o;
          o.x = pack2_ct(v[0], v[1]);
          o.y = pack2_ct(v[2], v[3]);
          *(uint2*)(ep + pw * ROWB + (((4 * i + g) ^ (pw & (NCK - 1))) << 4) + 8 * hw) = o;
        }
      }
#pragma unroll
      for (int q = 0; q < 32 / PPI; ++q) {
        const int p = lane / NCK + PPI * q, c = lane % NCK;
        const u32x4 val = *(const u32x4*)(ep + p * ROWB + ((c ^ (p & (NCK - 1))) << 4));
        const int tp = (pg * FW + j) * 32 + p;
        const int rho = (tp * cut.inv) >> 20, w = tp - rho * TW;   // tp / TW (tp < 1024)
        const int co = co0 + wc * MT * 32 + 8 * c;
        const int hv = h0 + rho, nz = TALL ? (hv * cut.invH) >> 20 : 0;
        if (rho < R && hv < Hv && w0 + w < W && co < Cout && (!TALL || hv - nz * cut.hp < H))
          *(u32x4*)(Yg + ((long)(n * H + hv - nz) * W + w0 + w) * Cout + co) = val;
      }
    }
  }
}

// y[p][co] = bf16(act(sum_{s < S} part[s][p][co] + b[co])), s ascending, of
// micro-batch blockIdx.y.
__global__ __launch_bounds__(256) void split_epilogue(TileIo io, const float* __restrict__ bias,
                                                      long n, int Cout, int S, int relu) {
  const long e = ((long)blockIdx.x * 256 + threadIdx.x) * 8;
  if (e >= n) return;
  const float* __restrict__ part = pickg(io.part, blockIdx.y);
  float v[8];
  const float4 a0 = *(const float4*)(part + e), a1 = *(const float4*)(part + e + 4);
  v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w;
  v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
  for (int s = 1; s < S; ++s) {
    const float4 b0 = *(const float4*)(part + (long)s * n + e);
    const float4 b1 = *(const float4*)(part + (long)s * n + e + 4);
    v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w;
    v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
  }
  const int co = e % Cout;
  u32x4 o;
#pragma unroll
  for (int t = 0; t < 8; t += 2) {
    float x0 = v[t], x1 = v[t + 1];
    if (bias) { x0 += bias[co + t]; x1 += bias[co + t + 1]; }
    if (relu) { x0 = fmaxf(x0, 0.f); x1 = fmaxf(x1, 0.f); }
    o[t / 2] = pack2_ct(x0, x1);
  }
  *(u32x4*)(pickg(io.y, blockIdx.y) + e) = o;
}

// Configurations, with what one round of blocks costs (measured in us: `a`
// per tile and `b` per 16-channel stage; 128 channels at 56 x 56 and 256 at
// 28 x 28, 32 samples).
struct TileCfg { int MT, WC, WP, FW, LW, NS; double a, b; };
constexpr TileCfg kTileCfgs[] = {
    {2, 2, 4, 2, 7, 2, 4.8, 2.0},    // 128 channels x 256 pixels
    {1, 2, 4, 4, 5, 3, 4.0, 1.94},   // 64 x 512
    {1, 2, 4, 2, 4, 4, 3.0, 1.2},    // 64 x 256
    {1, 2, 4, 1, 4, 4, 2.0, 0.8},    // 64 x 128
    {1, 1, 8, 2, 4, 4, 2.4, 1.07},   // 32 x 512
    {1, 1, 8, 1, 3, 4, 1.8, 0.69},   // 32 x 256
    {1, 1, 4, 1, 5, 3, 1.5, 0.5},    // 32 x 128, four waves
};
constexpr int kTileN = sizeof(kTileCfgs) / sizeof(kTileCfgs[0]);
// blocks of a configuration that a CU's 160 KiB of LDS hold
constexpr int tile_occ(const TileCfg& k) {
  return (k.NS * k.LW * k.WC * k.WP + k.NS + 1) * 2 <= 160 ? 2 : 1;
}

// The cut of an H x W image with the fewest tiles of at most px pixels whose
// R + 2 input rows fit `rows` LDS rows (the widest strips of those).
bool tile_cut(int H, int W, int px, int rows, TileCut& c) {
  long best = 0;
  for (int ns = 1; ns <= W; ++ns) {
    const int TW = (W + ns - 1) / ns;
    if (ns > 1 && TW < 8) break;
    const int BWP = (TW + 2 + 15) / 16 * 16;
    int R = px / TW;
    if (R > rows / BWP - 2) R = rows / BWP - 2;
    if (R > H) R = H;
    if (R < 1) continue;
    const int nrb = (H + R - 1) / R;
    const long tiles = (long)nrb * ((W + TW - 1) / TW);
    if (best == 0 || tiles < best) {
      best = tiles;
      R = (H + nrb - 1) / nrb;                    // even row blocks
      c = TileCut{R, TW, BWP, nrb, (W + TW - 1) / TW, ((1 << 20) + TW - 1) / TW,
                  ((1 << 20) + BWP - 1) / BWP, 0, 0};
    }
    if (TW <= 8) break;
  }
  return best > 0;
}

}  // namespace

thread_local int g_tile_cfg = -1;   // >= 0 forces a configuration (tests and measurement)

// Configurations that have a split-K form, and that have tiles across samples (for
// a sum split or not).
constexpr bool tile_splits(int c) { return c == 0 || c == 2 || c == 3; }
constexpr bool tile_tall(int c, int S) { return c == 3 || (c == 6 && S == 1); }

// Images of at most 64 pixels may share a tile: one sample to a tile of 128 leaves
// most of it idle (768 -> 640 at 3 x 3 x 12, four micro-batches, split sums, forward
// 86 -> 31 us; 576 -> 1152 at 2 x 2 x 13, two, 59 -> 19).
static bool tall_ok(const ConvShape& s) {
  return s.nb > 1 && s.H * s.W <= 64 && s.nb * (s.H + 1L) <= kTallRows;
}

// Configuration for ng micro-batches of a shape: the least estimated time,
// rounds of blocks times what a round costs.
static int tile_pick(const ConvShape& s, int ng, int S, TileCut& cut) {
  int best = -1;
  double best_cost = 0;
  const int nk = (s.cin + 15) / 16 / S;
  for (int c = 0; c < kTileN; ++c) {
    const TileCfg k = kTileCfgs[c];
    if (g_tile_cfg >= 0 && g_tile_cfg != c) continue;
    if (S > 1 && !tile_splits(c)) continue;
    const int NW = k.WC * k.WP, BN = 32 * k.MT * k.WC;
    for (int tall = 0; tall < 2; ++tall) {
      if (tall && !(tall_ok(s) && tile_tall(c, S))) continue;
      TileCut t;
      const int Hv = tall ? s.nb * (s.H + 1) - 1 : s.H;
      if (!tile_cut(Hv, s.W, 32 * k.WP * k.FW, k.LW * NW * 32 - 9 * BN, t)) continue;
      if (tall) {
        t.hp = s.H + 1;
        t.invH = ((1 << 20) + t.hp - 1) / t.hp;
      }
      const long items =
          (long)ng * (tall ? 1 : s.nb) * t.nrb * t.ns * ((s.cout + BN - 1) / BN) * S;
      const long rounds = (items + 255) / 256;
      const double cost = rounds * (k.a + nk * k.b) / (rounds > 1 && tile_occ(k) > 1 ? 1.4 : 1.0);
      if (best < 0 || cost < best_cost) {
        best = c;
        best_cost = cost;
        cut = t;
      }
    }
  }
  return best;
}

// Shares of a split sum, a function of the per-sample shape (so that every
// sample's sums keep their order whatever the micro-batch): two or four where
// four samples give few tiles of 64 x 256 and a share keeps 16 stages, of four 12.
// The shares' sums cost a write, a read and a launch (4 us), and more the more
// samples a launch has.  Forward with its epilogue, us, for 1, 2, 4 shares: 1024 at
// 14 x 14 x 1: 42, 32, 21; x 16: 80, 79, 86; 512 at 14 x 14 x 1: 23, 20, 15; 896 ->
// 192 at 7 x 7 x 1: 36, 26, 17; 896 -> 128 at 9 x 9 x 4: 37, 27, 18; 768 -> 128 at
// 17 x 17 x 32: 37, 39, 42; 256 at 16 x 16 x 1: 13, 14.  Images past 4096 pixels in
// four samples gain only with the longest sums (2048 -> 128 at 36 x 36 x 1: 80, 52;
// x 16: 101, 140).  Shares stop at 192 tiles, which bounds the room their sums
// take in a plan.
int conv_tile_split(const ConvShape& s) {
  const long P = 4L * s.H * s.W, nk = s.cin / 16;
  if (s.cin % 64 || s.cout % 64) return 1;
  const long tiles = (P + 255) / 256 * (s.cout / 64);
  if (P > 4096)
    return P <= 8192 && tiles <= 64 && s.cout % 128 == 0 && nk % 2 == 0 && nk / 2 >= 48 ? 2 : 1;
  int S = 1;
  while (S < 4 && tiles * S < 192 && nk / (2 * S) >= (S == 1 ? 16 : 12) && nk % (2 * S) == 0) S *= 2;
  return S;
}

bool conv_tile_ok(const ConvShape& s) {
  return s.taps == 9 && s.cin % 8 == 0 && s.cout % 8 == 0 && s.pixels() > 0 &&
         (double)s.pixels() * s.cin * 2 < 2147483648.0 &&
         (double)s.cout * 9 * s.cin * 2 < 2147483648.0;
}

template <int MT, int WC, int WP, int FW, int LW, int NS, bool DG, bool SPLIT, bool TALL = false>
static hipError_t launch_tile(const TileIo& io, int ng, const bf16_t* Wt, const float* b,
                              const ConvShape& s, int relu, int S, const TileCut& cut,
                              hipStream_t st) {
  static const KernelName name("conv3x3_tile<%d,%d,%d,%d,%d,%d%s%s%s>", MT, WC, WP, FW, LW, NS,
                               TALL ? ",tall" : "", DG ? ",dg" : "", SPLIT ? ",split" : "");
  constexpr int BN = 32 * MT * WC, NW = WC * WP;
  const long items = (long)ng * (TALL ? 1 : s.nb) * cut.nrb * cut.ns * ((s.cout + BN - 1) / BN) * S;
  constexpr int occ = tile_occ(TileCfg{MT, WC, WP, FW, LW, NS, 0, 0});
  const int G = (int)(items < 256 * occ ? items : 256 * occ);
  const long P = (long)ng * s.pixels();
  ProfScope ps(name.s, 2.0 * P * s.cout * 9 * s.cin,
               2.0 * ((double)P * s.cin + 9.0 * s.cin * s.cout + (double)P * s.cout), st);
  TGP_LAUNCH(ps, (conv3x3_tile<MT, WC, WP, FW, LW, NS, DG, SPLIT, TALL>), dim3(G), dim3(NW * 64), 0, st,
             io, ng, Wt, b, s.nb, s.H, s.W, s.cin, s.cout, relu, S, cut);
  return launch_status();
}

// y = act(conv(x, w) + b), or with dg the data gradient: x = dz, s the
// transposed shape (cin: its sum channels, the forward layer's outputs), and w
// the forward layer's weights.  With S > 1 (conv_tile_split) part[k] holds S
// nb H W Cout floats.
hipError_t conv_forward_tile(int n, const void* const* x, const void* w, const float* b,
                             void* const* y, const ConvShape& s, int relu, bool dg, int S,
                             float* const* part, hipStream_t st) {
  if (n < 1 || n > kMaxGroup || !conv_tile_ok(s) || !w || S < 1 || (S > 1 && !part))
    return hipErrorInvalidValue;
  if (n > kTileGroup) {
    for (int k0 = 0; k0 < n; k0 += kTileGroup) {
      const int c = n - k0 < kTileGroup ? n - k0 : kTileGroup;
      const hipError_t e =
          conv_forward_tile(c, x + k0, w, b, y + k0, s, relu, dg, S, S > 1 ? part + k0 : nullptr, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  TileCut cut{};
  const int c = tile_pick(s, n, S, cut);
  if (c < 0) return hipErrorInvalidValue;
  TileIo io{};
  for (int k = 0; k < kTileGroup; ++k) {   // unused entries repeat micro-batch 0
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.y[k] = (bf16_t*)y[k < n ? k : 0];
    io.part[k] = S > 1 ? part[k < n ? k : 0] : nullptr;
    if (!io.x[k] || !io.y[k] || (S > 1 && !io.part[k])) return hipErrorInvalidValue;
  }
  const bf16_t* Wt = (const bf16_t*)w;
#define CT_GO(i, D, SP)                                                                     \
  launch_tile<kTileCfgs[i].MT, kTileCfgs[i].WC, kTileCfgs[i].WP, kTileCfgs[i].FW,           \
              kTileCfgs[i].LW, kTileCfgs[i].NS, D, SP>(io, n, Wt, b, s, relu, S, cut, st)
#define CT_TALL(i, D, SP)                                                                   \
  launch_tile<kTileCfgs[i].MT, kTileCfgs[i].WC, kTileCfgs[i].WP, kTileCfgs[i].FW,           \
              kTileCfgs[i].LW, kTileCfgs[i].NS, D, SP, true>(io, n, Wt, b, s, relu, S, cut, st)
  if (S > 1) {
    hipError_t e = hipErrorInvalidValue;
    if (cut.hp) {
      if (c == 3) e = dg ? CT_TALL(3, true, true) : CT_TALL(3, false, true);
    } else switch (c) {
#define CT_CASE(i) \
  case i: e = dg ? CT_GO(i, true, true) : CT_GO(i, false, true); break;
      CT_CASE(0) CT_CASE(2) CT_CASE(3)
#undef CT_CASE
    }
    if (e != hipSuccess) return e;
    const long numel = s.pixels() * s.cout;
    ProfScope ps("split_epilogue", 0.0, n * numel * (4.0 * S + 2.0), st);
    TGP_LAUNCH(ps, split_epilogue, dim3((unsigned)((numel / 8 + 255) / 256), n), dim3(256), 0, st,
               io, b, numel, s.cout, S, relu);
    return launch_status();
  }
  if (cut.hp) {
    if (c == 3) return dg ? CT_TALL(3, true, false) : CT_TALL(3, false, false);
    if (c == 6) return dg ? CT_TALL(6, true, false) : CT_TALL(6, false, false);
    return hipErrorInvalidValue;
  }
  switch (c) {
#define CT_CASE(i) \
  case i: return dg ? CT_GO(i, true, false) : CT_GO(i, false, false);
    CT_CASE(0) CT_CASE(1) CT_CASE(2) CT_CASE(3) CT_CASE(4) CT_CASE(5) CT_CASE(6)
#undef CT_CASE
#undef CT_GO
#undef CT_TALL
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tgpk
