// Implicit-GEMM convolution / FC of few output rows on gfx950 matrix cores: small output
// tiles, operands straight from memory into registers, K splits inside the workgroup.
//
// At a handful of images a layer is a chain of latencies, not arithmetic: a 14 x 14 layer of
// one image has 196 rows, so the tiled kernel split its K over workgroups to fill the chip and
// a second launch added the partial sums (4.7 + 4.4 us for a 3x3 over 256 channels, of which
// a launch by itself is 2.6).  Here one workgroup owns a small output tile and its waves take
// the K splits: each wave streams its range of K through a ring of registers with no barrier,
// and the partial sums meet once, in LDS, in split order.  Layers that the shape leaves
// unsplit run one tile per wave.
//
// Tiles are 16 or 32 pixels x 16 or 32 channels (16x16x32 MFMAs): a tile of 16 x 16 loads as
// many bytes per compute unit as four K splits of a 64 x 128 tile and gives four to eight
// times the workgroups; the larger tiles halve the bytes where the rows suffice to fill the
// chip.  The tuner times them against the tiled kernel and its reduce launch.  ResNet-50's
// layers of one image (traced): 3x3 over 256 channels 4.7 + 4.4 -> 7 us, 3x3 over 512 channels
// 5.7 + 8.2 -> 12 us, 1x1 to 256 channels from 1024 4.6 + 4.0 -> 5.0 us; the whole model at one
// image takes 363 us without these tiles and 309 with them.  What is left is latency: the kernel arguments, one round of loads from
// the last-level cache, the meeting in LDS, the stores.  The first weights are requested before
// the pixel addresses are known, and the epilogue's operands before the K loop.
//
// Bits: v_mfma_f32_16x16x32_bf16 gives the sums of two v_mfma_f32_32x32x16_bf16 bit for
// bit, K runs in the packed order within a split, and the splits are those of the shape,
// added in order with the reduce kernel's epilogue.
#include "kernels.h"

namespace rafiki {

namespace {
typedef __bf16 bf16x8_s __attribute__((ext_vector_type(8)));
typedef float f32x4_s __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_s __attribute__((ext_vector_type(2)));
typedef float f32x2_s __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f_s(uint32_t b16) { return __uint_as_float(b16 << 16); }
__device__ __forceinline__ uint32_t f2bf_s(float f) {   // nearest, ties to even (finite)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}
// ReLU and rounding of two values as the launch that the tile stands for takes them: the reduce
// launch of a split K (fmaxf, which makes a NaN 0), or the unsplit tiled kernel (an integer max,
// which keeps a positive NaN, and the hardware's rounding).  Alike for every other value.
__device__ __forceinline__ uint32_t pack2_s(float a, float b, bool relu, bool split) {
  if (split) {
    if (relu) { a = fmaxf(a, 0.f); b = fmaxf(b, 0.f); }
    return f2bf_s(a) | (f2bf_s(b) << 16);
  }
  if (relu) {
    a = __int_as_float(max(__float_as_int(a), 0));
    b = __int_as_float(max(__float_as_int(b), 0));
  }
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_s{a, b}, bf16x2_s));
}
}  // namespace

// What the epilogue of one 16 x 16 block needs from memory, fetched before the K loop: the
// folded scale and shift of this lane's 4 channels c .. c + 3 and the residual of row m.
struct SmallFold {
  float4 sc, sh;
  uint2 res;
};
__device__ __forceinline__ SmallFold small_fold(const ConvArgs& a, int m, int c) {
  SmallFold f;
  f.sc = *(const float4*)(a.scale + c);   // c < Co_pad
  f.sh = *(const float4*)(a.shift + c);
  f.res = make_uint2(0u, 0u);
  if (a.res && !a.out_f32 && m < a.M && c + 4 <= a.c_write)
    f.res = *(const uint2*)((const bf16_t*)a.res + (long long)m * a.ldy + c);
  return f;
}
// One lane's 4 channels c .. c + 3 of GEMM row m: the epilogue of the split-K reduction, or
// (split false) of the unsplit tiled kernel.
// With the fused 2x2 max-pool the four rows of a window are four neighbouring lanes.
__device__ __forceinline__ void small_epilogue(const ConvArgs& a, f32x4_s acc, const SmallFold& f, int m, int c, bool split) {
  float v[4] = {acc[0] * f.sc.x + f.sh.x, acc[1] * f.sc.y + f.sh.y, acc[2] * f.sc.z + f.sh.z,
                acc[3] * f.sc.w + f.sh.w};
  if (a.pool2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = fmaxf(v[j], __shfl_xor(v[j], 1));
      v[j] = fmaxf(v[j], __shfl_xor(v[j], 2));
    }
    if ((m & 3) != 0) return;
    m >>= 2;
    if (m >= a.M / 4) return;
  } else if (m >= a.M) {
    return;
  }
  if (c >= a.c_write) return;
  const long long o = (long long)m * a.ldy + c;
  if (a.out_f32 || c + 4 > a.c_write) {   // fp32 rows (logits) of any stride, ragged channels
    for (int j = 0; j < 4; ++j) {
      if (c + j >= a.c_write) break;
      if (a.res) v[j] += bf2f_s(((const bf16_t*)a.res)[o + j]);
      const float t = a.relu ? fmaxf(v[j], 0.f) : v[j];
      if (a.out_f32) ((float*)a.y)[o + j] = t;
      else ((bf16_t*)a.y)[o + j] = (bf16_t)f2bf_s(t);
    }
    return;
  }
  if (a.res) {
    v[0] += bf2f_s(f.res.x & 0xFFFFu);
    v[1] += bf2f_s(f.res.x >> 16);
    v[2] += bf2f_s(f.res.y & 0xFFFFu);
    v[3] += bf2f_s(f.res.y >> 16);
  }
  uint2 p;
  p.x = pack2_s(v[0], v[1], a.relu, split);
  p.y = pack2_s(v[2], v[3], a.relu, split);
  *(uint2*)((bf16_t*)a.y + o) = p;
}

// x / d for x < 2^16 with mag = ceil(2^32 / d), or 0 for d = 1.
__device__ __forceinline__ int div_by(int x, unsigned mag) { return mag ? (int)__umulhi((unsigned)x, mag) : x; }

// Most waves of a workgroup: a 32 x 32 tile keeps up to 256 registers a wave.
constexpr int small_waves(int blocks) { return blocks >= 4 ? 8 : 16; }
// Magic divisors (div_by): pixel tiles, a map's rows of the GEMM, a map row, taps, a kernel row.
struct SmallMags {
  unsigned m_tiles, map, row, taps, kw;
};

template <int TMB, int TNB>
__global__ __launch_bounds__(small_waves(TMB * TNB) * 64) void conv_small_kernel(ConvArgs a, int splits, int m_tiles, SmallMags g) {
  use_member(a);
  // K tiles of 64 in flight per wave: 64 or 48 registers of a wave's 128 (16 waves), or 96 of 256
  constexpr int R = TMB * TNB == 1 ? 4 : (TMB * TNB == 2 ? 2 : 3);
  constexpr int NBLK = TMB * TNB;
  extern __shared__ f32x4_s small_part[];   // [waves][NBLK][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int r = lane & 15, kc = lane >> 4;
  // contiguous ranges of tiles per XCD, pixel tiles fastest: the tiles that share weights run
  // on one XCD, which fetches them into its L2 once
  const int G = gridDim.x, b = blockIdx.x;
  const int q = G >> 3, r8 = G & 7, xcd = b & 7, loc = b >> 3;
  const int blk = (xcd < r8 ? xcd * (q + 1) : r8 * (q + 1) + (xcd - r8) * q) + loc;
  const int tile = splits == 1 ? blk * nw + wave : blk;
  const int nt = div_by(tile, g.m_tiles), mt = tile - nt * m_tiles;
  if (splits == 1 && nt >= a.n_tiles) return;   // no barrier on this path
  const int m0 = mt * 16 * TMB, n0 = nt * 16 * TNB;

  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, (short)0, a.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, (short)0, a.w_bytes, 0x00020000);
  constexpr unsigned kOob = 0xFFFFFF00u;   // past every buffer: the hardware returns zeros
  unsigned woff[TNB];
#pragma unroll
  for (int t = 0; t < TNB; ++t) woff[t] = (unsigned)(((n0 + t * 16 + r) * a.Kp + kc * 8) * 2);

  const int taps = a.kh * a.kw, ktiles = a.Kp / 64;
  bf16x8_s xb[R][TMB][2], wb[R][TNB][2];
  f32x4_s acc[TMB][TNB];
  f32x4_s sum = {};   // of this wave's block (wave < NBLK) over all splits so far
  static_assert(NBLK <= small_waves(NBLK), "one block per wave at most");
  auto wload = [&](int i, int kt, bool live) {
#pragma unroll
    for (int t = 0; t < TNB; ++t) {
      const unsigned off = live ? woff[t] + (unsigned)kt * 128u : kOob;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wb[i][t][h] = __builtin_bit_cast(bf16x8_s, __builtin_amdgcn_raw_buffer_load_b128(wr, (int)(off + 64 * h), 0, 0));
    }
  };
  // this wave's split of round s0: its first K tile and K tiles
  auto first_of = [&](int s0) { return (splits == 1 ? 0 : s0 + wave) * a.kt_per_split; };
  auto count_of = [&](int s0) {
    return splits == 1 || s0 + wave < splits ? min(a.kt_per_split, ktiles - first_of(s0)) : 0;
  };
  // the first weights are on their way while the pixel addresses are computed
#pragma unroll
  for (int i = 0; i < R; ++i) wload(i, first_of(0) + i, i < count_of(0));
  
  int hi0[TMB], wi0[TMB], xoff[TMB];
#pragma unroll
  for (int t = 0; t < TMB; ++t) {
    const int m = m0 + t * 16 + r;
    int n, ho, wo;
    if (a.pool2) {   // row m: position m % 4 of 2x2 window m / 4
      const int w4 = m >> 2, Wo2 = a.Wo >> 1, HW2 = (a.Ho >> 1) * Wo2;
      n = div_by(w4, g.map);
      const int rem = w4 - n * HW2, ho2 = div_by(rem, g.row);
      ho = 2 * ho2 + ((m >> 1) & 1);
      wo = 2 * (rem - ho2 * Wo2) + (m & 1);
    } else {
      n = div_by(m, g.map);
      const int rem = m - n * (a.Ho * a.Wo);
      ho = div_by(rem, g.row);
      wo = rem - ho * a.Wo;
    }
    hi0[t] = m < a.M ? ho * a.stride - a.pad : -(1 << 28);
    wi0[t] = wo * a.stride - a.pad;
    xoff[t] = m < a.M ? (((n * a.H + hi0[t]) * a.W + wi0[t]) * a.Cs + kc * 8) * 2 : 0;
  }

  // one block's worth at most: an unsplit tile of several blocks would not keep them in registers
  SmallFold fold;
  if (NBLK == 1 || (splits > 1 && wave < NBLK)) {
    const int k = splits > 1 ? wave % NBLK : 0;
    fold = small_fold(a, m0 + k / TNB * 16 + r, n0 + k % TNB * 16 + 4 * kc);
  }

  for (int s0 = 0; s0 < splits; s0 += nw) {
    const int kt0 = first_of(s0), nk = count_of(s0);
    // K tile kt0 + k is channel block cb at tap (u, v)
    int cb = div_by(kt0, g.taps);
    const int tap0 = kt0 - cb * taps;
    int u = div_by(tap0, g.kw), v = tap0 - u * a.kw;
    auto xload = [&](int i, bool live) {
      const int delta = ((u * a.W + v) * a.Cs + cb * 64) * 2;
#pragma unroll
      for (int t = 0; t < TMB; ++t) {
        const bool ok = live && (unsigned)(hi0[t] + u) < (unsigned)a.H && (unsigned)(wi0[t] + v) < (unsigned)a.W;
        const unsigned off = ok ? (unsigned)(xoff[t] + delta) : kOob;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          xb[i][t][h] = __builtin_bit_cast(bf16x8_s, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(off + 64 * h), 0, 0));
      }
      if (++v == a.kw) {
        v = 0;
        if (++u == a.kh) {
          u = 0;
          ++cb;
        }
      }
    };
    auto mfmas = [&](int i) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int tn = 0; tn < TNB; ++tn)
#pragma unroll
          for (int tm = 0; tm < TMB; ++tm)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[i][tn][h], xb[i][tm][h], acc[tm][tn], 0, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int j = 0; j < TNB; ++j) acc[i][j] = f32x4_s{0.f, 0.f, 0.f, 0.f};
    if (s0 > 0) {
#pragma unroll
      for (int i = 0; i < R; ++i) wload(i, kt0 + i, i < nk);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) xload(i, i < nk);
    int k = 0;
    for (; k + R < nk; k += R) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        mfmas(i);
        // past the range: out-of-bounds offsets, no memory traffic
        wload(i, kt0 + k + i + R, k + i + R < nk);
        xload(i, k + i + R < nk);
      }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (k + i < nk) mfmas(i);
    if (splits == 1) {
#pragma unroll
      for (int b = 0; b < NBLK; ++b) {
        const int m = m0 + b / TNB * 16 + r, c = n0 + b % TNB * 16 + 4 * kc;
        small_epilogue(a, acc[b / TNB][b % TNB], NBLK == 1 ? fold : small_fold(a, m, c), m, c, false);
      }
      return;
    }
    if (s0 > 0) __syncthreads();   // the previous round's sums have been read
#pragma unroll
    for (int tm = 0; tm < TMB; ++tm)
#pragma unroll
      for (int tn = 0; tn < TNB; ++tn) small_part[(wave * NBLK + tm * TNB + tn) * 64 + lane] = acc[tm][tn];
    __syncthreads();
    if (wave < NBLK) {
      const int here = min(nw, splits - s0);
      for (int k = 0; k < here; ++k) {
        const f32x4_s p = small_part[(k * NBLK + wave) * 64 + lane];
        if (s0 + k == 0) sum = p;
        else sum += p;
      }
    }
  }
  if (wave < NBLK) small_epilogue(a, sum, fold, m0 + wave / TNB * 16 + r, n0 + wave % TNB * 16 + 4 * kc,
                                  true);
}

bool conv_small_fits(const ConvArgs& a, int tile) {
  if (tile < 0 || tile >= kNumSmallTiles) return false;
  const long long tm = kSmallTiles[tile][0], tn = kSmallTiles[tile][1];
  const long long tiles = (a.M + tm - 1) / tm * (((a.c_write > a.Nc ? a.c_write : a.Nc) + tn - 1) / tn);
  return a.Cs % 64 == 0 && a.tap_stride == 0 && !a.tok && !a.maxslot && a.Kp == a.K && a.M > 0 && a.Nc > 0 &&
         a.M + 64 < 1 << 16 && tiles + 16 < 1 << 16;   // div_by's range
}

const int kSmallTiles[kNumSmallTiles][2] = {{16, 16}, {16, 32}, {32, 16}, {32, 32}};

hipError_t launch_conv_small(const ConvArgs& a0, int tile, int splits, hipStream_t s) {
  ConvArgs a = a0;
  if (splits < 1 || !conv_small_fits(a, tile) || a.n_members > kMaxGroup)
    return hipErrorInvalidValue;
  const int tm = kSmallTiles[tile][0], tn = kSmallTiles[tile][1], nblk = tm * tn / 256;
  const int m_tiles = (a.M + tm - 1) / tm;
  // every written channel (storage padding included); rows past Nc are zero weights up to Co_pad
  a.n_tiles = ((a.c_write > a.Nc ? a.c_write : a.Nc) + tn - 1) / tn;
  // waves: over the splits in equal rounds, at least one per 16 x 16 block of the tile
  int nw = 4;
  if (splits > 1) {
    const int most = small_waves(nblk), rounds = (splits + most - 1) / most;
    nw = (splits + rounds - 1) / rounds;
    if (nw < nblk) nw = nblk;
  }
  const int tiles = m_tiles * a.n_tiles, blocks = splits > 1 ? tiles : (tiles + nw - 1) / nw;
  const dim3 grid((unsigned)blocks, 1, a.n_members > 1 ? a.n_members : 1), block(nw * 64);
  const size_t lds = splits > 1 ? (size_t)nw * nblk * 64 * 16 : 0;
  auto mag = [](int d) { return d == 1 ? 0u : (unsigned)((((unsigned long long)1 << 32) + d - 1) / d); };
  const int map = a.pool2 ? (a.Ho / 2) * (a.Wo / 2) : a.Ho * a.Wo;
  const SmallMags g{mag(m_tiles), mag(map), mag(a.pool2 ? a.Wo / 2 : a.Wo), mag(a.kh * a.kw), mag(a.kw)};
  const LaunchEvents& ev = launch_events();
#define RAFIKI_SMALL(T, M, N)                                                                                     \
  case T:                                                                                                         \
    if (ev.start || ev.stop)                                                                                      \
      hipExtLaunchKernelGGL((conv_small_kernel<M, N>), grid, block, lds, s, ev.start, ev.stop, 0, a, splits, m_tiles, g); \
    else                                                                                                          \
      hipLaunchKernelGGL((conv_small_kernel<M, N>), grid, block, lds, s, a, splits, m_tiles, g);                     \
    break;
  switch (tile) {
    RAFIKI_SMALL(0, 1, 1) RAFIKI_SMALL(1, 1, 2) RAFIKI_SMALL(2, 2, 1) RAFIKI_SMALL(3, 2, 2)
  }
#undef RAFIKI_SMALL
  return hipGetLastError();
}

}  // namespace rafiki
