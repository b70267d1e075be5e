// 3x3 stride-1 convolution of many channels on gfx950 matrix cores, from an LDS patch and
// streamed weights: VGG-16's layers of 128 to 512 channels.
//
// The tiled GEMM brings both operands into LDS for every 64 terms of K and meets at a barrier
// each time: its fragment reads (6 KB per wave for 8 MFMAs) and LDS writes alone take the time
// of its MFMAs, and it ran these layers at 0.38 to 0.42 of the bf16 peak.  Here
//  - the nine taps of a block of 64 channels read one patch of the input (the tile's pixels and
//    their halo), so pixels enter LDS once per block and there is one barrier per 576 terms; the
//    next block's patch travels in registers meanwhile;
//  - every weight is used by one wave (or two), so weights skip LDS: they lie in memory in the
//    order of use and stream through a ring of registers, six steps of 32 terms ahead;
//  - a wave computes 128 pixels x 64 channels, one wave per SIMD: 8 KB of LDS reads and 4 KB of
//    weights for 16 MFMAs, 64 and 32 bytes a cycle per compute unit, half of what either path
//    delivers.
//
// A workgroup of 4 waves computes 128 pixels x 256 channels (one group of pixels, four of
// channels) or 256 x 128 (two by two).  Its pixels are consecutive in NHWC (FLAT: the patch is one
// contiguous run of pixels and a lane masks the taps outside the image) or a rectangle 16 or 32
// pixels wide (the patch holds zeros outside the image).  Rectangles leave part of a tile idle on
// maps they do not divide, but hold whole 2x2 windows, with a window's rows in one lane and its
// columns in two neighbouring lanes, for the fused max-pool.
//
// Everything in the main loop is issued between MFMAs (the step's comment): 86 % of its cycles
// are MFMAs, 43 k of a tile's 55 k cycles at 256 channels; patch, epilogue and stores of a tile
// take the rest, with nothing on the compute unit to hide them, and the clock falls to 1.8 GHz
// under the load.  VGG-16 at 64 images (traced, tiled GEMM before): conv3_2 229 -> 194 us
// (1,220 TFLOP/s), conv4_2 230 -> 199, conv5_1 70 -> 52, conv2_2 with its pool 250 -> 221.
// Without the interleaving 239, 213, 217 and 57.
//
// Bits: K in the packed order (channel block, tap, channel), the GEMM's MFMA and operand roles,
// epilogue fma(acc, scale, shift) (max over the window), ReLU, one rounding.
#include "kernels.h"

namespace rafiki {

namespace {
typedef __bf16 bf16x8_p __attribute__((ext_vector_type(8)));
typedef float f32x16_p __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_p __attribute__((ext_vector_type(2)));
typedef float f32x2_p __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack2_p(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_p{a, b}, bf16x2_p));
}
__device__ __forceinline__ float relu_p(float v) { return __int_as_float(max(__float_as_int(v), 0)); }
__device__ __forceinline__ void lds_barrier_p() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// LDS rows of 64 channels (8 chunks of 16 bytes): row r keeps chunk c at slot c ^ psw(r); 16 lanes
// reading one chunk of 16 consecutive rows touch every bank once.
__device__ __forceinline__ int psw(int r) { return (r >> 1) & 7; }
}  // namespace

// MODE 0: consecutive pixels; 16, 32: rectangles that wide.
template <int WPX, int MODE, bool POOL>
__global__ __launch_bounds__(256, 1) void conv_patch_kernel(ConvArgs a) {
  constexpr int WCH = 4 / WPX;                 // wave grid: WPX groups of 128 pixels x WCH of 64 channels
  constexpr int BM = 128 * WPX, BN = 64 * WCH;
  constexpr bool FLAT = MODE == 0;
  constexpr int TW = FLAT ? 1 : MODE, TH = BM / TW;
  constexpr int PROWS = FLAT ? kPatchFlatRows : (TH + 2) * (TW + 2);
  constexpr int NLD = (PROWS * 8 + 255) / 256;
  constexpr int R = 6;                         // steps of 32 terms in flight; 18 steps per channel block
  static_assert(!(FLAT && POOL), "a window's rows are apart in consecutive pixels");
  constexpr int STG = 4 * 128 * 8;             // epilogue: 128 rows x 64 channels of bf16 per wave
  __shared__ uint4 lds[(2 * PROWS * 8 > STG ? 2 * PROWS * 8 : STG) + 8];
  constexpr int ZEROB = (2 * PROWS * 8 > STG ? 2 * PROWS * 8 : STG) * 16;   // 128 zero bytes

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wp = wave % WPX, wc = wave / WPX;
  const int frow = lane & 31, fk = lane >> 5;
  const int G = gridDim.x, b = blockIdx.x;
  const int q = G >> 3, r8 = G & 7, xcd = b & 7, loc = b >> 3;
  const int tile = (xcd < r8 ? xcd * (q + 1) : r8 * (q + 1) + (xcd - r8) * q) + loc;
  const int nt = tile % a.n_tiles, mt = tile / a.n_tiles;
  const int n0 = nt * BN;
  // FLAT: first pixel m0.  Rectangles: image img, top-left (h0, w0).
  int m0 = 0, img = 0, h0 = 0, w0 = 0;
  if constexpr (FLAT) {
    m0 = mt * BM;
  } else {
    const int tx = (a.W + TW - 1) / TW, ty = (a.H + TH - 1) / TH;
    img = mt / (tx * ty);
    const int rem = mt - img * (tx * ty);
    h0 = rem / tx * TH;
    w0 = rem % tx * TW;
  }
  const int npx = a.N * a.H * a.W;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, (short)0, a.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, (short)0, a.w_bytes, 0x00020000);

  // ---- this thread's part of a patch: LDS chunk i * 256 + tid
  unsigned poff[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int it = i * 256 + tid, r = it >> 3, c = (it & 7) ^ psw(r);
    bool ok;
    int px;
    if constexpr (FLAT) {
      px = m0 - a.W - 1 + r;
      ok = r < BM + 2 * (a.W + 1) && px >= 0 && px < npx;
    } else {
      const int pr = r / (TW + 2), pc = r - pr * (TW + 2), h = h0 - 1 + pr, w = w0 - 1 + pc;
      px = (img * a.H + h) * a.W + w;
      ok = r < PROWS && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
    }
    // outside: an offset past the buffer (and stays past it as the channel block is added)
    poff[i] = ok ? (unsigned)px * (unsigned)(a.Cs * 2) + c * 16 : 0x80000000u;
  }
  uint4 pv[NLD];
  auto pload = [&](int cb) {
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      pv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)poff[i], cb * 128, 0));
  };
  auto pstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      if (i * 256 + tid < PROWS * 8) lds[buf * (PROWS * 8) + i * 256 + tid] = pv[i];
  };
  const int ncb = a.Cs / 64;
  pload(0);
  // ---- weight ring: 4 KB per step for this wave's 64 channels
  const int wlane = lane * 16;
  int wofs = (n0 / 64 + wc) * (ncb * 18 * 4096);
  const int wlast = wofs + (ncb * 18 - 1) * 4096;
  bf16x8_p wf[R][2][2];   // [step][channel block of 32][16 terms]
  auto wload = [&](int i) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
      wf[i][h >> 1][h & 1] =
          __builtin_bit_cast(bf16x8_p, __builtin_amdgcn_raw_buffer_load_b128(wr, wlane + h * 1024, wofs, 0));
    wofs = min(wofs + 4096, wlast);   // past the last step: the last again, not used
  };
#pragma unroll
  for (int i = 0; i < R - 1; ++i) wload(i);

  // ---- this lane's pixels: block t of 32
  int prow[4];       // patch row of tap (0, 0)
  unsigned mask[4];  // FLAT: the taps inside the image
  const int PW = FLAT ? a.W : TW + 2;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if constexpr (FLAT) {
      const int i = wp * 128 + t * 32 + frow, m = m0 + i;
      const int w = m % a.W, h = (m / a.W) % a.H;
      unsigned v = 0;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int hh = h + k / 3 - 1, ww = w + k % 3 - 1;
        if (m < npx && (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W) v |= 1u << k;
      }
      mask[t] = v;
      prow[t] = i;
    } else {
      // rows of a window in blocks t and t + 1 (t even), its columns in neighbouring lanes
      const int pr = wp * (128 / TW) + (TW == 16 ? 2 * (2 * (t >> 1) + (frow >> 4)) + (t & 1) : t);
      prow[t] = pr * PW + (frow & (TW - 1));
      mask[t] = 0x1FF;
    }
  }
  if (tid < 8) lds[ZEROB / 16 + tid] = make_uint4(0u, 0u, 0u, 0u);
  pstore(0);
  lds_barrier_p();

  const char* const ldsb = (const char*)lds;
  int ad[4];
  bf16x8_p xf[2][4][2];
  auto address = [&](int buf, int tap, int toff) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int r = prow[t] + toff;
      const int at = buf * (PROWS * 128) + r * 128 + ((psw(r) ^ fk) << 4);
      ad[t] = !FLAT || ((mask[t] >> tap) & 1u) ? at : ZEROB + (fk << 4);
    }
  };
  auto frags = [&](bf16x8_p (&x)[4][2], int half) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) x[t][h] = *(const bf16x8_p*)(ldsb + (ad[t] ^ ((half * 4 + h * 2) << 4)));
  };
  f32x16_p acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  for (int cb = 0; cb < ncb; ++cb) {
    const int buf = cb & 1;
    if (cb + 1 < ncb) pload(cb + 1);
    address(buf, 0, 0);
    frags(xf[0], 0);
    int tap = 0, tv = 0, toff = 0;
    for (int g = 0; g < 3; ++g) {   // three taps (a kernel row) per round of the ring
#pragma unroll
      for (int i = 0; i < R; ++i) {
        wload((i + R - 1) % R);   // the slot that the previous step used
        if ((i & 1) == 0) {
          frags(xf[1], 1);
        } else {
          ++tap;   // the next tap (after the last: its own addresses again, not used)
          if (++tv == 3) {
            tv = 0;
            toff += PW - 2;
          } else {
            ++toff;
          }
          if (tap < 9) address(buf, tap, toff);
          frags(xf[0], 0);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int t = 0; t < 4; ++t)
              acc[tn][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][tn][h], xf[i & 1][t][h], acc[tn][t], 0, 0, 0);
        // One wave per SIMD: whatever is not issued between MFMAs (32 cycles each) is time the
        // matrix core idles.  The next step's addresses, then its 8 fragment reads, then the 4
        // weight loads, one after each MFMA.
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // MFMA
          if (k < 4) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);       // VALU
          else if (k < 12) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); // LDS read
          else __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);             // memory read
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (cb + 1 < ncb) pstore(buf ^ 1);
    lds_barrier_p();   // the next patch is visible, and every wave is done with this one
  }

  // ---- epilogue: rounded outputs staged per wave as [128 pixels][64 channels] (or the 32 pooled
  // pixels), then whole 128-byte rows per pixel
  uint4* const stg = lds + wave * (128 * 8);
#pragma unroll
  for (int tn = 0; tn < 2; ++tn)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = n0 + wc * 64 + tn * 32 + 8 * g + 4 * fk;
      const float4 sc = *(const float4*)(a.scale + c);
      const float4 sh = *(const float4*)(a.shift + c);
      float v[4][4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v[t][0] = acc[tn][t][4 * g + 0] * sc.x + sh.x;
        v[t][1] = acc[tn][t][4 * g + 1] * sc.y + sh.y;
        v[t][2] = acc[tn][t][4 * g + 2] * sc.z + sh.z;
        v[t][3] = acc[tn][t][4 * g + 3] * sc.w + sh.w;
      }
      if constexpr (POOL) {
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
          float m[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            m[j] = fmaxf(v[t][j], v[t + 1][j]);
            m[j] = fmaxf(m[j], __shfl_xor(m[j], 1));
            if (a.relu) m[j] = relu_p(m[j]);
          }
          // pooled pixel of blocks t, t + 1 and lane pair frow / 2
          const int r = (t >> 1) * 16 + (frow >> 1);
          if ((frow & 1) == 0)
            *((uint2*)(stg + r * 8 + ((4 * tn + g) ^ psw(r))) + fk) = make_uint2(pack2_p(m[0], m[1]), pack2_p(m[2], m[3]));
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = t * 32 + frow;
          if (a.relu) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[t][j] = relu_p(v[t][j]);
          }
          *((uint2*)(stg + r * 8 + ((4 * tn + g) ^ psw(r))) + fk) =
              make_uint2(pack2_p(v[t][0], v[t][1]), pack2_p(v[t][2], v[t][3]));
        }
      }
    }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  const int oct = lane & 7;
#pragma unroll
  for (int p = 0; p < (POOL ? 4 : 16); ++p) {
    const int r = p * 8 + (lane >> 3);
    long long m;   // output row, or -1
    if constexpr (FLAT) {
      const int i = m0 + wp * 128 + r;
      m = i < npx ? i : -1;
    } else if constexpr (POOL) {
      // pooled row / column of the wave's rectangle
      const int pr = wp * (64 / TW) + (TW == 16 ? 2 * (r >> 4) + ((r >> 3) & 1) : r >> 4);
      const int h = h0 / 2 + pr, w = w0 / 2 + (TW == 16 ? r & 7 : r & 15);
      m = h < a.H / 2 && w < a.W / 2 ? ((long long)img * (a.H / 2) + h) * (a.W / 2) + w : -1;
    } else {
      const int t = r >> 5, f = r & 31;
      const int pr = wp * (128 / TW) + (TW == 16 ? 2 * (2 * (t >> 1) + (f >> 4)) + (t & 1) : t);
      const int h = h0 + pr, w = w0 + (f & (TW - 1));
      m = h < a.H && w < a.W ? ((long long)img * a.H + h) * a.W + w : -1;
    }
    if (m >= 0)
      *(uint4*)((bf16_t*)a.y + m * a.ldy + n0 + wc * 64 + 8 * oct) = stg[r * 8 + (oct ^ psw(r))];
  }
}

// The weights [Co][Kp] of a 3x3 layer in conv_patch_kernel's order: per group of 64 channels and
// step of 32 terms, four fragments (channel blocks of 32 x 16 terms) of 64 lanes x 8 terms.
__global__ void pack_patch_weights_kernel(const bf16_t* w, int kp, int steps, bf16_t* out, long long total) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = (int)(idx & 63), h = (int)(idx >> 6) & 1, tn = (int)(idx >> 7) & 1;
  const long long gs = idx >> 8;
  const int g = (int)(gs / steps), s = (int)(gs - (long long)g * steps);
  const int row = g * 64 + tn * 32 + (lane & 31), k = s * 32 + h * 16 + 8 * (lane >> 5);
  *(uint4*)(out + idx * 8) = *(const uint4*)(w + (size_t)row * kp + k);
}

hipError_t launch_pack_patch_weights(const bf16_t* w, int kp, int co, int K, bf16_t* out, hipStream_t s) {
  const long long total = (long long)co * K / 8;
  launch(pack_patch_weights_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), s, w, kp, K / 32, out, total);
  return hipGetLastError();
}

bool conv_patch_fits(const ConvArgs& a, int cfg) {
  const bool wide = a.Nc % 256 == 0;
  if (cfg < 0 || cfg >= kNumPatchTiles) return false;
  const int mode = kPatchModes[cfg];
  if (a.kh != 3 || a.kw != 3 || a.stride != 1 || a.pad != 1 || a.Ho != a.H || a.Wo != a.W || a.Cs % 64 != 0 ||
      a.Nc % 128 != 0 || a.c_write != a.Nc || a.ldy != a.Nc || a.K != 9 * a.Cs || a.Kp != a.K || a.res || a.out_f32 ||
      a.n_members > 1 || a.tap_stride != 0 || a.tok || a.maxslot)
    return false;
  if (a.pool2 && (mode == 0 || a.H % 2 != 0 || a.W % 2 != 0)) return false;
  if (mode == 0) return wide && 128 + 2 * (a.W + 1) <= kPatchFlatRows;
  return wide || mode == 16;
}

const int kPatchModes[kNumPatchTiles] = {0, 16, 32};

#define RAFIKI_PATCH(X) X(1, 0, false) X(1, 16, false) X(1, 16, true) X(1, 32, false) X(1, 32, true) X(2, 16, false) X(2, 16, true)
#define RAFIKI_INST(P, M, PO) template __global__ void conv_patch_kernel<P, M, PO>(ConvArgs);
RAFIKI_PATCH(RAFIKI_INST)
#undef RAFIKI_INST

hipError_t launch_conv_patch(const ConvArgs& a0, const void* w, int cfg, hipStream_t s) {
  if (!conv_patch_fits(a0, cfg)) return hipErrorInvalidValue;
  ConvArgs a = a0;
  const int mode = kPatchModes[cfg], wpx = a.Nc % 256 == 0 ? 1 : 2, bm = 128 * wpx, bn = 256 / wpx;
  a.w = w;
  a.w_bytes = a.Nc * a.K * 2;
  a.n_tiles = a.Nc / bn;
  const long long px = (long long)a.N * a.H * a.W;
  const int th = mode ? bm / mode : 0;
  const long long tiles = mode ? (long long)a.N * ((a.W + mode - 1) / mode) * ((a.H + th - 1) / th) : (px + bm - 1) / bm;
  const dim3 grid((unsigned)(tiles * a.n_tiles));
#define RAFIKI_CASE(P, M, PO)                                                    \
  if (wpx == P && mode == M && (a.pool2 != 0) == PO) {                           \
    launch((conv_patch_kernel<P, M, PO>), grid, dim3(256), s, a);                \
    return hipGetLastError();                                                    \
  }
  RAFIKI_PATCH(RAFIKI_CASE)
#undef RAFIKI_CASE
  return hipErrorInvalidValue;
}
#undef RAFIKI_PATCH

}  // namespace rafiki
