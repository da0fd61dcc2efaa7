// bf16 3x3 weight gradient for any image size and any channel counts that
// are multiples of 8, on 32 x 32 x 16 MFMA with operands read from LDS by the
// gfx950 transpose loads.
//
// dW[co][r][s][ci] = sum_p dZ[p][co] X[p + (r - 1) W + (s - 1)][ci].  A work
// item is (K range, 64 output channels, 64 input channels) with all nine
// taps.  The twelve waves of a block, three per SIMD, are (filter row, 32
// input channels, phase of k steps); each accumulates 64 output x 32 input
// channels for the three column taps of its filter row over every other k
// step of 16 pixels, two dZ and three input fragments feeding six MFMAs.  (A
// 32 x 32 wave tile reads four fragments for three MFMAs: LDS then takes
// longer than the MFMAs, and the kernel ran 1.2 to 1.5 times longer.)  The
// two phases' sums meet through LDS at the end of an item.
//
// An item's K range is a run of stages; a stage is RPS rows x TW columns of
// one sample (the image is cut into column strips so that a stage fills its
// LDS slot).  A stage holds the dZ pixels, each image row padded to a
// multiple of 8 pixels, and the RPS + 2 input rows, each a block of BW =
// padded width + 4 LDS rows whose first and TW + 1st pixels are the halo.  LDS rows are 64 channels (128
// bytes), their 16-byte chunks XOR-swizzled by 2 (row & 3).  A k step is two
// units of 8 pixels, each within one image row, so the half-waves take their
// own row's offset.  Pixels outside the image, channels past Cin or Cout and
// the padding are buffer reads at out-of-range offsets (zeros); the input of
// a unit's padding pixels (past the strip's real width, which for the last
// strip may end in any unit of a row) is also cleared in registers, since it
// may be a real pixel that no output pairs with that tap, or unset LDS, and 0 x
// Inf is not 0.  Rows past the image are not summed at all.
//
// Each item writes its fp32 slice for its K range; the slices are summed in
// K-range order.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {


// Barrier between LDS writes and other waves' reads of them (or the other way
// round): this wave's LDS accesses have completed when it arrives, and the
// compiler moves none across it.
__device__ __forceinline__ void wt_handoff() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The micro-batches of one launch (nb samples each); micro-batch k's slices
// go to out[k].  A larger group runs as launches of eight.
constexpr int kWtGroup = 8;
struct WtIo {
  const bf16_t* x[kWtGroup];
  const bf16_t* dz[kWtGroup];
  float* out[kWtGroup];
};
// Stage geometry: RPS rows x TW columns, n8 units of 8 pixels per row, AROWS
// LDS rows of dZ, nrb row blocks and ns strips per sample, T stages per
// micro-batch in nK ranges of spk; invT = ceil(2^20 / (8 n8)), invB =
// ceil(2^20 / (8 n8 + 4)) (exact quotients for the LDS rows of a slot).
struct WtCut {
  int RPS, TW, n8, AROWS, nrb, ns, T, nK, spk, invT, invB;
};

constexpr int kWtNW = 12;    // waves
template <int LW, int NS>
__global__ __launch_bounds__(64 * kWtNW) void conv_wgrad_tile(WtIo io, int ng, int nb, int H, int W,
                                                              int Cin, int Cout, WtCut cut) {
  constexpr int NW = kWtNW;
  constexpr int SB = LW * NW * 1024;            // slot bytes
  // The last k step of an odd count of units reads its second unit from the
  // rows after the stage's input (and clears it): up to the first 8 pixels and
  // 2 column taps of the next row, which may lie past the last slot.
  constexpr int TAIL = (8 + 2) * 128;
  static_assert(NS * SB + TAIL <= 160 * 1024, "LDS ring");
  static_assert(6 * 12 * 1024 <= SB, "exchange of the phases' sums fits a slot");
  __shared__ __attribute__((aligned(16))) unsigned char smem[NS * SB + TAIL];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = wave >> 2;                     // filter row
  const int nw = wave & 1, ph = wave >> 1 & 1;  // input half, phase of k steps
  const int n8 = cut.n8, TWP = 8 * n8, BW = TWP + 4;
  const int nct = (Cout + 63) / 64, ncit = (Cin + 63) / 64;
  const int per_k = nct * ncit;                 // items per K range
  const int items = ng * cut.nK * per_k;
  const int G = gridDim.x;
  const int lb = xcd_remap(blockIdx.x, G);
  const int n_items = lb < items ? (items - lb + G - 1) / G : 0;
  const long E = (long)Cout * 9 * Cin;
  const int zbytes = nb * H * W * Cout * 2, xbytes = nb * H * W * Cin * 2;

  // DMA lane constants: instruction u of this wave fills chunk c = NW u +
  // wave, LDS rows 8 c + lane / 8, physical 16-byte chunk lane % 8, which
  // holds logical chunk lc.  Rows below AROWS are dZ pixels, the rest input.
  const int lc = (lane & 7) ^ (2 * ((lane >> 3) & 3));
  int doff[LW], drc[LW];                        // byte offset; row | column << 16, or -1
#pragma unroll
  for (int u = 0; u < LW; ++u) {
    const int c = NW * u + wave;
    const int row = c * 8 + (lane >> 3);
    if (c * 8 < cut.AROWS) {
      const int pr = (row * cut.invT) >> 20, pc = row - pr * TWP;   // row / TWP
      const bool ok = pr < cut.RPS && pc < cut.TW;
      doff[u] = ok ? ((pr * W + pc) * Cout + 8 * lc) * 2 : 0;
      drc[u] = ok ? pr | (pc << 16) : -1;
    } else {
      const int q = row - cut.AROWS;
      const int rr = (q * cut.invB) >> 20, cc = q - rr * BW;        // q / BW
      const bool ok = rr < cut.RPS + 2 && cc < cut.TW + 2;
      doff[u] = ok ? ((rr * W + cc - 1) * Cin + 8 * lc) * 2 : 0;
      drc[u] = ok ? rr | (cc << 16) : -1;
    }
  }

  // Fragment lane constants (byte offsets in a stage).  Lane group g = lane /
  // 16 holds MFMA rows / columns 16 (g % 2) .. + 15 and k 8 (g / 2) .. + 7;
  // lane j = lane % 16 addresses pixel k + j / 4, channels + 4 (j % 4).
  const int g = lane >> 4, j = lane & 15, half = lane >> 5;
  const int kb = 8 * (g >> 1) + (j >> 2);
  const int cha = (16 * (g & 1) + 4 * (j & 3)) * 2;
  const int chb = (nw * 32 + 16 * (g & 1) + 4 * (j & 3)) * 2;
  int fa[2];                                    // the two 32-channel halves
#pragma unroll
  for (int i = 0; i < 2; ++i)
    fa[i] = kb * 128 + (((4 * i + (cha >> 4)) ^ (2 * (kb & 3))) << 4) + (cha & 15);
  int fb[3];
#pragma unroll
  for (int s = 0; s < 3; ++s)
    fb[s] = cut.AROWS * 128 + fr * BW * 128 + (kb + s) * 128 +
            (((chb >> 4) ^ (2 * ((kb + s) & 3))) << 4) + (chb & 15);

  auto coords = [&](int it, int& kr, int& co0, int& ci0) __attribute__((always_inline)) {
    const int item = lb + it * G;
    kr = item / per_k;
    const int t = item - kr * per_k;
    co0 = (t / ncit) * 64;
    ci0 = (t % ncit) * 64;
  };
  // K range kr's first stage and stage count within its micro-batch
  auto range_of = [&](int kr, int& s0) __attribute__((always_inline)) {
    s0 = (kr % cut.nK) * cut.spk;
    return min(cut.spk, cut.T - s0);
  };

  int i_it = 0, i_st = 0, i_s0 = 0, i_n = 0, i_co0 = 0, i_ci0 = 0;
  u32x4 rzg = {}, rxg = {};
  auto issue_item = [&]() __attribute__((always_inline)) {
    int kr;
    coords(i_it, kr, i_co0, i_ci0);
    i_n = range_of(kr, i_s0);
    const int gi = kr / cut.nK;
    rzg = make_rsrc(pickg(io.dz, gi), zbytes);
    rxg = make_rsrc(pickg(io.x, gi), xbytes);
  };
  if (n_items > 0) issue_item();
  auto issue = [&](int slot) __attribute__((always_inline)) {
    const int st = i_s0 + i_st;                 // stage: (sample, strip, row block)
    const int col = st / cut.nrb;
    const int h = (st - col * cut.nrb) * cut.RPS;
    const int n = col / cut.ns, w0 = (col - n * cut.ns) * cut.TW;
    const int zb = (((n * H + h) * W + w0) * Cout + i_co0) * 2;
    const int xb = (((n * H + h - 1) * W + w0) * Cin + i_ci0) * 2;   // negative above the image
    const bool zc = i_co0 + 8 * lc < Cout, xc = i_ci0 + 8 * lc < Cin;
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int c = NW * u + wave;
      auto* dst = TGP_LDS(smem + slot * SB + c * 1024);
      const int r = drc[u] & 0xffff, cc = drc[u] >> 16;
      if (c * 8 < cut.AROWS) {                  // wave-uniform
        const bool ok = drc[u] >= 0 && zc && h + r < H && w0 + cc < W;
        dma16(rzg, dst, ok ? doff[u] + zb : kOob, 0);
      } else {
        const bool ok = drc[u] >= 0 && xc && (unsigned)(h - 1 + r) < (unsigned)H &&
                        (unsigned)(w0 + cc - 1) < (unsigned)W;
        dma16(rxg, dst, ok ? doff[u] + xb : kOob, 0);
      }
    }
    if (++i_st == i_n) {
      i_st = 0;
      if (++i_it < n_items) issue_item();
    }
  };

  // four units per k step of a phase: rows and units of a row they advance
  const int step_r = 4 / n8, step_u = 4 - step_r * n8;
  int total = 0;
  for (int it = 0; it < n_items; ++it) {
    int kr, co0, ci0, s0;
    coords(it, kr, co0, ci0);
    total += range_of(kr, s0);
  }
#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < total) issue(k);

  int idx = 0;
  for (int c_it = 0; c_it < n_items; ++c_it) {
    int kr, co0, ci0, s0;
    coords(c_it, kr, co0, ci0);
    const int ns = range_of(kr, s0);
    f32x16_t acc[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s = 0; s < 3; ++s) acc[i][s] = f32x16_t{};
    for (int st = 0; st < ns; ++st, ++idx) {
      wait_stages<NS, LW>(min(NS - 2, total - 1 - idx));
      ring_barrier();
      // The slot freed last stage is refilled at once.  (One instruction per k
      // step between the MFMAs was 20 to 60% slower; half the waves issuing
      // theirs in mid-stage, with the next step's fragments loaded behind the
      // MFMAs, 30%.)
      if (idx + NS - 1 < total) issue((idx + NS - 1) % NS);
      const unsigned char* sp = smem + (idx % NS) * SB;
      const int sg = s0 + st, col = sg / cut.nrb;
      const int h = (sg - col * cut.nrb) * cut.RPS;
      const int w0 = (col - (col / cut.ns) * cut.ns) * cut.TW;
      const int U = min(cut.RPS, H - h) * n8;   // units of this stage
      const int KT = (U + 1) / 2;
      const int tw = min(cut.TW, W - w0);       // pixels of a row
      const int ul = (tw - 1) >> 3;             // unit that holds its last one, as pixel rem - 1
      const int rem = tw - 8 * ul;
      const bool ragged = tw < TWP || (U & 1);  // some unit has padding pixels
      unsigned mrem[4];                         // rem pixels of a fragment's 8
#pragma unroll
      for (int e = 0; e < 4; ++e)
        mrem[e] = (rem > 2 * e ? 0xffffu : 0u) | (rem > 2 * e + 1 ? 0xffff0000u : 0u);
      // this half-wave's unit: its index in the row, and the extra LDS rows of
      // its image row's block (4 per row)
      int uc = half + 2 * ph, ue = (uc / n8) * (4 * 128);
      uc -= (uc / n8) * n8;
      for (int t = ph; t < KT; t += 2) {
        u32x4 a[2], b[3];
        const int ka = 16 * t * 128;
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = frag_tr(sp + fa[i] + ka, 128);
#pragma unroll
        for (int s = 0; s < 3; ++s) b[s] = frag_tr(sp + fb[s] + ka + ue, 128);
        // units with padding pixels: unit ul of a row (rem real ones), and past
        // it or past an odd count (none); skipped by the waves that have none
        const bool pad = 2 * t + half >= U || uc > ul;
        if (ragged && __any(pad || uc == ul)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const unsigned m = pad ? 0u : uc == ul ? mrem[e] : ~0u;
#pragma unroll
            for (int s = 0; s < 3; ++s) b[s][e] &= m;
          }
        }
        uc += step_u;
        ue += step_r * (4 * 128);
        if (uc >= n8) { uc -= n8; ue += 4 * 128; }
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i][s] = mfma32(as_bf16x8(a[i]), as_bf16x8(b[s]), acc[i][s]);
      }
    }
    // the phases meet in the slot of the stage just consumed (free once every
    // wave is past its last reads; its refill is issued only after the next
    // stage's barrier): phase 0 gets the first 32 output channels, phase 1
    // the second, each sum phase 0 + phase 1
    ring_barrier();
    f32x4_t* const xs = (f32x4_t*)(smem + ((idx - 1) % NS) * SB) + (2 * fr + nw) * 12 * 64 + lane;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (i) wt_handoff();
      if (ph != i) {
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            xs[(4 * s + q) * 64] = f32x4_t{acc[i][s][4 * q], acc[i][s][4 * q + 1],
                                           acc[i][s][4 * q + 2], acc[i][s][4 * q + 3]};
      }
      wt_handoff();
      if (ph == i) {
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4_t v = xs[(4 * s + q) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][s][4 * q + e] += v[e];
          }
      }
    }
    // epilogue: element v of lane l of acc[i][s] is co 32 i + 8 (v / 4) + 4 (l
    // / 32) + v % 4, ci l % 32 of this wave's channels, tap (fr, s)
    const int gi = kr / cut.nK;
    float* o = pickg(io.out, gi) + (long)(kr - gi * cut.nK) * E;
    const int ci = ci0 + nw * 32 + (lane & 31);
    if (ci < Cin) {
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int co = co0 + 32 * ph + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          if (co < Cout)
            o[((long)co * 9 + 3 * fr + s) * Cin + ci] = ph ? acc[1][s][v] : acc[0][s][v];
        }
    }
  }
}

constexpr int kWtLW = 6, kWtNS = 2;             // 72 KiB slots, two stages
constexpr int kWtRows = kWtLW * kWtNW * 8;      // LDS rows of a slot

// The stage geometry of a micro-batch and its K ranges.
//  - Strips and rows: the fewest 16-pixel k steps per image, a stage's fixed
//    cost counting as kStageSteps of them; fewer rows where the micro-batch
//    has too few stages for kItems items, but not more than two stages for each
//    range it may have (below 256 pixels that is one, and its stages a chain: 24
//    -> 16 channels at 6 x 4, ten samples, stages of one row 62 us).
//  - K ranges: about kItems items per micro-batch (a launch over four then
//    fills two rounds of blocks; one micro-batch alone runs on half the CUs),
//    at most 8 MB of slices (their write and re-read otherwise cost more than
//    the parallelism gains) and no more slices than the general kernels
//    write, so that a plan needs no more room than with those.  A function of one micro-batch's shape, so a
//    group gives the bits of single launches.
constexpr double kStageSteps = 4.0;
constexpr int kItems = 128;
WtCut wt_cut(const ConvShape& s) {
  const long per_k = (long)((s.cout + 63) / 64) * ((s.cin + 63) / 64);
  const long E = (long)s.cout * 9 * s.cin;
  const long kmax = std::min({(kItems + per_k - 1) / per_k, std::max(1L, (8L << 20) / (4 * E)),
                              (long)wgrad_general_splits(s)});
  WtCut best{};
  double best_cost = 0;
  for (int ns = 1; ns <= s.W; ++ns) {
    const int TW = ns == 1 ? s.W : ((s.W + ns - 1) / ns + 7) / 8 * 8, n8 = (TW + 7) / 8;
    if (ns > 1 && TW < 16) break;
    const int nst = (s.W + TW - 1) / TW;
    const long rows = s.nb * (long)nst * s.H;
    const int maxr = (int)std::min((long)s.H, std::max({1L, rows * per_k / kItems, rows / (2 * kmax)}));
    int RPS = 0;
    while (RPS < s.H && RPS < maxr &&
           (((RPS + 1) * n8 + 1) / 2) * 16 + (RPS + 3) * (8 * n8 + 4) <= kWtRows)
      ++RPS;
    if (RPS < 1) continue;
    const int nrb = (s.H + RPS - 1) / RPS;
    RPS = (s.H + nrb - 1) / nrb;                // even row blocks
    const double cost = (double)nst * nrb * (((RPS * n8 + 1) / 2) + kStageSteps);
    if (best.RPS && cost >= best_cost) continue;
    best_cost = cost;
    best = WtCut{RPS, TW, n8, ((RPS * n8 + 1) / 2) * 16, nrb, nst, s.nb * nst * nrb, 1, 0,
                 ((1 << 20) + 8 * n8 - 1) / (8 * n8), ((1 << 20) + 8 * n8 + 3) / (8 * n8 + 4)};
  }
  const long nK = std::min(kmax, (long)best.T);
  best.spk = (int)((best.T + nK - 1) / nK);
  best.nK = (best.T + best.spk - 1) / best.spk;
  return best;
}

}  // namespace

bool wgrad_tile_ok(const ConvShape& s) {
  return s.taps == 9 && s.cin % 8 == 0 && s.cout % 8 == 0 && s.pixels() > 0 &&
         (double)s.pixels() * (s.cin > s.cout ? s.cin : s.cout) * 2 < 2147483648.0;
}

double wgrad_tile_fill(const ConvShape& s) {
  const WtCut c = wt_cut(s);
  return (double)s.pixels() / ((double)c.T * c.AROWS);
}

size_t wgrad_tile_partial_floats(const ConvShape& s) {
  const int S = wt_cut(s).nK;
  return S > 1 ? (size_t)S * s.cout * 9 * s.cin : 0;
}

// n (1 .. kMaxGroup) micro-batches in one launch, each sum left pending in
// *defer[k].
hipError_t conv_wgrad_tile_launch(int n, const void* const* x, const void* const* dz,
                                  float* const* dw, float* const* partial, const ConvShape& s,
                                  hipStream_t st, ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup || !wgrad_tile_ok(s)) return hipErrorInvalidValue;
  if (n > kWtGroup) {
    for (int k0 = 0; k0 < n; k0 += kWtGroup) {
      const int c = n - k0 < kWtGroup ? n - k0 : kWtGroup;
      const hipError_t e =
          conv_wgrad_tile_launch(c, x + k0, dz + k0, dw + k0, partial + k0, s, st, defer + k0);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const WtCut c = wt_cut(s);
  WtIo io{};
  for (int k = 0; k < kWtGroup; ++k) {   // unused entries repeat micro-batch 0
    const int q = k < n ? k : 0;
    io.x[k] = (const bf16_t*)x[q];
    io.dz[k] = (const bf16_t*)dz[q];
    io.out[k] = c.nK > 1 ? partial[q] : dw[q];
    if (!io.x[k] || !io.dz[k] || !io.out[k] || !defer[q]) return hipErrorInvalidValue;
  }
  const long E = (long)s.cout * 9 * s.cin;
  const long items = (long)n * c.nK * ((s.cout + 63) / 64) * ((s.cin + 63) / 64);
  const int G = (int)(items < 256 ? items : 256);
  {
    ProfScope ps("conv_wgrad_tile", 2.0 * n * s.pixels() * E,
                 n * (2.0 * s.pixels() * (s.cin + s.cout) + 4.0 * c.nK * E), st);
    TGP_LAUNCH(ps, (conv_wgrad_tile<kWtLW, kWtNS>), dim3(G), dim3(64 * kWtNW), 0, st, io, n, s.nb,
               s.H, s.W, s.cin, s.cout, c);
  }
  const hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{io.out[k], dw[k], E, c.nK};
  return hipSuccess;
}

}  // namespace tgpk
