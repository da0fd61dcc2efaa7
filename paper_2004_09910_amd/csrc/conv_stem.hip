// bf16 3x3 convolution of few input channels (1 .. 7: an image) into any
// multiple of 8 output channels, and its weight gradient, on 32 x 32 x 16 MFMA.
//
// The sum has 9 Cin <= 63 terms, so both are one or two thin products whose
// other operand, the output (or its gradient), is what has to move: they are
// bound by writing Y and reading dZ once.  The im2col operand is never laid
// out: each lane gathers its 8 terms of a pixel (forward) or its 8 pixels of a
// term (weight gradient) by 2-byte buffer loads, whose out-of-range offsets
// give the zeros of the padding.  Measured at 3 -> 64, 192 x 192 x 4 (us): forward 46
// on the float32 matrix unit -> 14, weight gradient 234 -> 19.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_util.h"
#include "prof.h"

namespace tgpk {
namespace {

struct StemIo {
  const bf16_t* x[kMaxGroup];
  bf16_t* y[kMaxGroup];
  const bf16_t* dz[kMaxGroup];
  float* out[kMaxGroup];
};


// Input tensors may start at any even address: a descriptor's base is the
// 4-byte word the tensor starts in, `lead` (0 or 2) the bytes before it.
struct StemX {
  __amdgpu_buffer_rsrc_t r;
  int lead;
};
__device__ __forceinline__ StemX stem_x(const bf16_t* x, int bytes) {
  const unsigned long a = (unsigned long)x;
  const int lead = (int)(a & 2);
  return {__builtin_amdgcn_make_buffer_rsrc((void*)(a - lead), 0, bytes + lead, 0x00020000), lead};
}
__device__ __forceinline__ unsigned ld_u16(const StemX& x, int voff, bool ok) {
  return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(x.r, ok ? voff + x.lead : kOob, 0, 0);
}
__device__ __forceinline__ bf16x8_t pack8(const unsigned (&v)[8]) {
  return as_bf16x8(u32x4{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16});
}
// Taps inside the image of pixel p (bit 3 r + s); none past the end.
__device__ __forceinline__ unsigned tap_mask(int p, int P, int H, int W) {
  if (p >= P) return 0;
  const unsigned q = (unsigned)p / (unsigned)W;
  const int w = p - (int)q * W, h = (int)(q % (unsigned)H);
  const unsigned cols = (w > 0 ? 1u : 0u) | 2u | (w + 1 < W ? 4u : 0u);
  return (h > 0 ? cols : 0u) | cols << 3 | (h + 1 < H ? cols << 6 : 0u);
}
// Term k < 64 of the sum: (tap, channel); its byte offset from the pixel.
// `inv` is 1024 / Cin + 1: k inv / 1024 = k / Cin, as k / 1024 < 1 / Cin.
__device__ __forceinline__ void term(int k, int W, int Cin, int inv, int& off, int& tap) {
  tap = k * inv >> 10;
  off = (((tap / 3 - 1) * W + tap % 3 - 1) * Cin + k - tap * Cin) * 2;
  if (tap > 8) tap = 31;                                        // no bit of a mask
}

// A wave's item is 32 pixels x 64 output channels, NB blocks of 16 terms; its
// outputs pass through LDS so that each store instruction writes 1 KB in a row.
template <int NB>
__global__ __launch_bounds__(256) void stem_fwd(StemIo io, int ng, const bf16_t* __restrict__ Wt,
                                                const float* __restrict__ bias, int P, int H, int W,
                                                int Cin, int Cout, int relu) {
  constexpr int PITCH = 144;                                    // 64 channels + 16 bytes
  __shared__ __attribute__((aligned(16))) unsigned char tile[4][32 * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h8 = 8 * (lane >> 5), l31 = lane & 31;
  const int co0 = blockIdx.y * 64, K = 9 * Cin, inv = 1024 / Cin + 1;
  // This tile's weights through LDS, in 2-byte steps of their own order (read
  // row by row by each lane, every load touches 64 cache lines).
  unsigned short* const ws = (unsigned short*)&tile[0][0];
  const int nw = min(64, Cout - co0) * K;
  for (int e = tid; e < nw; e += 256) ws[e] = ((const unsigned short*)Wt)[(long)co0 * K + e];
  __syncthreads();
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void*)bias, 0, bias ? Cout * 4 : 0, 0x00020000);
  bf16x8_t wf[2][NB];
  int off[NB][8], tap[NB][8];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int j = 0; j < 8; ++j) term(16 * b + h8 + j, W, Cin, inv, off[b][j], tap[b][j]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int co = co0 + 32 * i + l31;
      unsigned v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = 16 * b + h8 + j;
        const int e = (32 * i + l31) * K + k;
        v[j] = ws[k < K && co < Cout ? e : 0];
        if (k >= K || co >= Cout) v[j] = 0;
      }
      wf[i][b] = pack8(v);
    }
  }
  float bv[2][16];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int co = co0 + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      bv[i][v] = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(rb, co < Cout ? co * 4 : kOob, 0, 0));
    }
  __syncthreads();                                              // ws is read
  const int npt = (P + 31) / 32, items = ng * npt;
  unsigned char* const tw = tile[wave];
  for (int it = blockIdx.x * 4 + wave; it < items; it += gridDim.x * 4) {
    const int g = __builtin_amdgcn_readfirstlane(it / npt), p0 = (it - g * npt) * 32;
    const StemX rx = stem_x(pickg(io.x, g), P * Cin * 2);
    const int p = p0 + l31;
    const unsigned m = tap_mask(p, P, H, W);
    unsigned v[NB][8];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[b][j] = ld_u16(rx, p * Cin * 2 + off[b][j], (m >> tap[b][j]) & 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f32x16_t acc = f32x16_t{};
#pragma unroll
      for (int b = 0; b < NB; ++b) acc = mfma32(wf[i][b], pack8(v[b]), acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = acc[4 * q + e] + bv[i][4 * q + e];
          if (relu) o[e] = fmaxf(o[e], 0.f);
        }
        *(uint2*)(tw + l31 * PITCH + 64 * i + 16 * q + h8) =
            make_uint2(f2bf(o[0]) | f2bf(o[1]) << 16, f2bf(o[2]) | f2bf(o[3]) << 16);
      }
    }
    // same wave's LDS: in order, no barrier
    bf16_t* const y = pickg(io.y, g);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 8 * u + (lane >> 3), co = co0 + 8 * (lane & 7);
      const uint4 o = *(const uint4*)(tw + r * PITCH + 16 * (lane & 7));
      if (p0 + r < P && co < Cout) *(uint4*)(y + (long)(p0 + r) * Cout + co) = o;
    }
  }
}

// An item is (K range of 64-pixel stages, 64 output channels) x all terms (NT
// tiles of 32).  The NW waves of a block take a range's stages in turn, each
// with an LDS stage of its own (64 dZ rows of 128 bytes, chunks swizzled by
// 2 (row & 3)), and are added in wave order at the end: a plan has room for at
// most 64 ranges, so a block has to keep a CU's worth of loads in flight.
template <int NT, int NW>
__global__ __launch_bounds__(64 * NW) void stem_wgrad(StemIo io, int ng, int P, int H, int W,
                                                      int Cin, int Cout, int nK, int spk) {
  constexpr int SB = 8192 * NT;                                 // per wave: a stage, then its sums
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * SB];
  __shared__ __attribute__((aligned(16))) unsigned short masks[NW][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = __builtin_amdgcn_readfirstlane(blockIdx.x / nK);
  const int kr = blockIdx.x - g * nK, co0 = blockIdx.y * 64, K = 9 * Cin;
  const int T = (P + 63) / 64, s1 = min(T, (kr + 1) * spk);
  unsigned char* const sp = smem + wave * SB;
  const u32x4 rz = make_rsrc(pickg(io.dz, g), P * Cout * 2);
  const StemX rx = stem_x(pickg(io.x, g), P * Cin * 2);
  int off[NT], tap[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) term(32 * t + (lane & 31), W, Cin, 1024 / Cin + 1, off[t], tap[t]);
  const int rl = lane >> 3, ch = co0 + 8 * ((lane & 7) ^ (2 * (rl & 3)));
  // transposed fragment: lane group lane / 16 holds channels 16 (group % 2) ..
  // + 15, pixels 8 (group / 2) .. + 7
  const int kb = 8 * (lane >> 5) + ((lane & 15) >> 2);
  int fa[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int cb = (i * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
    fa[i] = kb * 128 + (((cb >> 4) ^ (2 * (kb & 3))) << 4) + (cb & 15);
  }
  f32x16_t acc[2][NT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[i][t] = f32x16_t{};

  for (int s = kr * spk + wave; s < s1; s += NW) {
    const int p0 = s * 64;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the last stage is read
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int p = p0 + 8 * u + rl;
      dma16(rz, TGP_LDS(sp + u * 1024), p < P && ch < Cout ? (p * Cout + ch) * 2 : kOob, 0);
    }
    masks[wave][lane] = (unsigned short)tap_mask(p0 + lane, P, H, W);
    unsigned v[4][NT][8];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int q0 = 16 * kk + 8 * (lane >> 5);
      const uint4 m4 = *(const uint4*)&masks[wave][q0];
      const unsigned mw[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const unsigned m = (mw[j >> 1] >> (16 * (j & 1))) & 0xffff;
          v[kk][t][j] = ld_u16(rx, (p0 + q0 + j) * Cin * 2 + off[t], (m >> tap[t]) & 1);
        }
    }
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      bf16x8_t a[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = as_bf16x8(frag_tr(sp + fa[i] + kk * 16 * 128, 128));
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const bf16x8_t b = pack8(v[kk][t]);
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][t] = mfma32(a[i], b, acc[i][t]);
      }
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // sums of the waves, in wave order: [channel][term] of 32 NT floats
  float* const mine = (float*)sp;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        mine[(32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 32 * NT + 32 * t + (lane & 31)] =
            acc[i][t][e];
  __syncthreads();
  float* const o = pickg(io.out, g) + (long)kr * Cout * K;
  for (int e = tid; e < 64 * 32 * NT; e += 64 * NW) {
    const int co = co0 + e / (32 * NT), k = e % (32 * NT);
    float r = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) r += ((const float*)(smem + w * SB))[e];
    if (co < Cout && k < K) o[(long)co * K + k] = r;
  }
}

// K ranges: as many as a plan has room for, at least one stage a wave.
struct StemCut { int nK, spk; };
StemCut stem_cut(const ConvShape& s) {
  const long T = (s.pixels() + 63) / 64, E = (long)s.cout * 9 * s.cin;
  const long nK = std::max(1L, std::min({(T + 15) / 16, std::max(1L, (8L << 20) / (4 * E)),
                                         (long)direct_wgrad_splits(s.pixels())}));
  const int spk = (int)((T + nK - 1) / nK);
  return {(int)((T + spk - 1) / spk), spk};
}

}  // namespace

bool conv_stem_ok(int dt, const ConvShape& s) {
  return dt == 0 && s.taps == 9 && s.cin >= 1 && s.cin <= 7 && s.cout % 8 == 0 && s.cout > 0 &&
         s.pixels() > 0 && (double)s.pixels() * s.cout * 2 < 2147483648.0 - 65536;
}

hipError_t conv_stem_forward(int n, const void* const* x, const void* w, const float* b,
                             void* const* y, const ConvShape& s, int relu, hipStream_t st) {
  if (n < 1 || n > kMaxGroup || !conv_stem_ok(0, s)) return hipErrorInvalidValue;
  StemIo io{};
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    io.x[k] = (const bf16_t*)x[k < n ? k : 0];
    io.y[k] = (bf16_t*)y[k < n ? k : 0];
  }
  const long P = s.pixels(), items = n * ((P + 31) / 32);
  if (items >= (1L << 31) - 8192) return hipErrorInvalidValue;
  // two items a wave, which share its weights; one where that leaves CUs idle (6 ->
  // 16 channels at 40 x 12: 10.6 -> 8.1 us)
  const long per = items < 1024 ? 4 : 8;
  const dim3 grid((unsigned)std::min(1024L, (items + per - 1) / per), (unsigned)((s.cout + 63) / 64));
  const bf16_t* Wt = (const bf16_t*)w;
  ProfScope ps("conv_stem", 2.0 * n * P * s.cout * 9 * s.cin, 2.0 * n * P * (s.cin + s.cout), st);
#define STEM_GO(NB) \
  TGP_LAUNCH(ps, stem_fwd<NB>, grid, dim3(256), 0, st, io, n, Wt, b, (int)P, s.H, s.W, s.cin, s.cout, relu)
  switch ((9 * s.cin + 15) / 16) {
    case 1: STEM_GO(1); break;
    case 2: STEM_GO(2); break;
    case 3: STEM_GO(3); break;
    default: STEM_GO(4);
  }
#undef STEM_GO
  return launch_status();
}

size_t conv_stem_wgrad_partial_floats(const ConvShape& s) {
  const int S = stem_cut(s).nK;
  return S > 1 ? (size_t)S * s.cout * 9 * s.cin : 0;
}

// n micro-batches in one launch, each sum left pending in *defer[k].
hipError_t conv_stem_wgrad_launch(int n, const void* const* x, const void* const* dz,
                                  float* const* dw, float* const* partial, const ConvShape& s,
                                  hipStream_t st, ReduceJob* const* defer) {
  if (n < 1 || n > kMaxGroup || !conv_stem_ok(0, s)) return hipErrorInvalidValue;
  const StemCut c = stem_cut(s);
  StemIo io{};
  for (int k = 0; k < kMaxGroup; ++k) {   // unused entries repeat the first
    const int q = k < n ? k : 0;
    io.x[k] = (const bf16_t*)x[q];
    io.dz[k] = (const bf16_t*)dz[q];
    io.out[k] = c.nK > 1 ? partial[q] : dw[q];
  }
  const long E = (long)s.cout * 9 * s.cin;
  const dim3 grid((unsigned)(n * c.nK), (unsigned)((s.cout + 63) / 64));
  {
    ProfScope ps("conv_stem_wgrad", 2.0 * n * s.pixels() * E,
                 n * (2.0 * s.pixels() * (s.cin + s.cout) + 4.0 * c.nK * E), st);
    if (9 * s.cin <= 32)
      TGP_LAUNCH(ps, (stem_wgrad<1, 16>), grid, dim3(1024), 0, st, io, n, (int)s.pixels(), s.H, s.W,
                 s.cin, s.cout, c.nK, c.spk);
    else
      TGP_LAUNCH(ps, (stem_wgrad<2, 8>), grid, dim3(512), 0, st, io, n, (int)s.pixels(), s.H, s.W,
                 s.cin, s.cout, c.nK, c.spk);
  }
  const hipError_t e = launch_status();
  if (e != hipSuccess) return e;
  for (int k = 0; k < n; ++k) *defer[k] = ReduceJob{io.out[k], dw[k], E, c.nK};
  return hipSuccess;
}

}  // namespace tgpk
