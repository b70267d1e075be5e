// Fused bottleneck block on gfx950 matrix cores: the 3x3 convolution, the 1x1 expansion
// with its residual and, where the next block follows directly, that block's 1x1
// reduction, for one tile of output pixels per workgroup and in one launch.
//
// Run apart, the three layers of a 14 x 14 block at 64 images took 26 + 20 + 15 us, a
// quarter of the matrix rate: each launch filled the chip for a short K, brought every
// pixel operand into LDS once per tap and per channel tile, and stored a tensor that the
// next launch read back.  Here a workgroup keeps its tile: the input patch (the tile's
// pixels and the rows above and below, contiguous in NHWC) is read into LDS once and the
// nine taps read it in place; the 3x3 output stays in LDS; the expansion runs in chunks of
// MID channels, each stored as the block's output and at once used as a slice of K of the
// next reduction.
//
// Every weight is used by exactly one wave of the workgroup (wave w owns channels
// 32 w .. 32 w + 31 of each chunk), so weights skip LDS: they lie in memory in the order
// in which the wave consumes them (pack_block_weights_kernel), 2 KB per 32 terms of K, and
// stream through a ring of registers that runs on across the phases.  A step of 32 terms is
// four 32x32x16 MFMAs per 64 pixels; per compute unit it needs 128 bytes a cycle from LDS
// and, with 64 pixels a tile, 64 bytes a cycle of weights from L2, both at their rates,
// which is why the tile is not smaller where the launch fills the chip.
//
// Bits: each output sums its K terms in the order of the layer-by-layer kernels with the
// same MFMA, including their split-K partial sums (summed in split order), the same
// epilogue fma(acc, scale, shift) (+ residual), ReLU (NaNs as in those kernels) and one
// rounding to bf16.
#include "kernels.h"

namespace rafiki {

namespace {
typedef __bf16 bf16x8_b __attribute__((ext_vector_type(8)));
typedef float f32x16_b __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2_b __attribute__((ext_vector_type(2)));
typedef float f32x2_b __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_b __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f_b(uint32_t b16) { return __uint_as_float(b16 << 16); }
__device__ __forceinline__ uint32_t pack2_b(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_b{a, b}, bf16x2_b));
}
__device__ __forceinline__ float relu_b(float v) { return __int_as_float(max(__float_as_int(v), 0)); }
// A NaN as a negative one, which relu_b makes 0.
__device__ __forceinline__ float negative_nan(float v) { return v == v ? v : __uint_as_float(0xFFC00000u); }

// Every wave's LDS accesses are done, then all waves pass.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void lds_wave_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}
}  // namespace

// LDS rows of MID channels (MID / 8 chunks of 16 bytes): row r keeps chunk c at slot
// c ^ rsw(r), so that 16 lanes reading one chunk of 16 consecutive rows touch every bank
// once (a row of at least 256 bytes starts at bank 0; 128-byte rows alternate halves).
template <int MID>
__device__ __forceinline__ int rsw(int r) {
  return MID >= 128 ? (r & 15) : ((r >> 1) & 7);
}

template <int MID, int BM, bool HASB, bool HASA>
__global__ __launch_bounds__(MID * 2, 2) void block_kernel(BlockArgs a) {
  constexpr int NW = MID / 32;          // waves
  constexpr int D = MID / 32;           // steps of 32 terms per K = MID; depth of the weight ring
  constexpr int NCH = MID / 8;          // 16-byte chunks per row
  constexpr int TP = BM / 32;           // 32-pixel blocks
  constexpr int NB = HASB ? 9 * D : 0;  // steps of the 3x3
  constexpr int WM = kBlockRowBytes / MID;   // widest map whose patch fits
  constexpr int PR = HASB ? BM + 2 * (WM + 1) : 0;
  constexpr int XROWS = PR > BM ? PR : BM;   // patch, later one expansion chunk
  constexpr int TAB = MID * (HASB ? 1 : 0) + 4 * MID + (HASA ? MID : 0);
  static_assert(D >= 2 && D % 2 == 0, "a tap is two steps");
  __shared__ uint4 lds[XROWS * NCH + BM * NCH + 8 + TAB / 2];
  uint4* const xbuf = lds;                       // [XROWS][NCH]
  uint4* const mid = lds + XROWS * NCH;          // [BM][NCH]
  uint4* const zero = mid + BM * NCH;            // 128 zero bytes
  float* const tab = (float*)(zero + 8);         // scale and shift of each phase

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int frow = lane & 31, fk = lane >> 5;
  // contiguous ranges of tiles per XCD: neighbouring tiles share patch rows in its L2
  const int G = gridDim.x, b = blockIdx.x;
  const int q = G >> 3, r8 = G & 7, xcd = b & 7, loc = b >> 3;
  const int tile = (xcd < r8 ? xcd * (q + 1) : r8 * (q + 1) + (xcd - r8) * q) + loc;
  const int m0 = tile * BM;

  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, (short)0, a.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, (short)0, a.w_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)a.res, (short)0, a.y_bytes, 0x00020000);

  // ---- input rows: the patch of the 3x3 (pixels m0 - W - 1 .. m0 + BM + W), or the tile
  constexpr int IN_ROWS = HASB ? PR : BM;
  constexpr int NLD = (IN_ROWS * NCH + NW * 64 - 1) / (NW * 64);
  uint4 pv[NLD];
  const int halo = HASB ? a.W + 1 : 0;
  const int rows = BM + 2 * halo;
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int it = i * (NW * 64) + tid;
    const int r = it / NCH, c = (it % NCH) ^ rsw<MID>(r);
    const int px = m0 - halo + r;
    // rows outside the tensor: an offset past the buffer, which reads zeros
    const unsigned off = r < rows && px >= 0 && px < a.M ? (unsigned)(px * NCH + c) * 16u : 0xFFFFFFF0u;
    pv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)off, 0, 0));
  }
  // ---- weight ring: the first D steps
  const int wlane = lane * 16;
  int wofs = wave * a.w_wave_bytes;   // next step's bytes
  bf16x8_b wf[D][2];
  auto wload = [&](int i) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      wf[i][h] = __builtin_bit_cast(bf16x8_b, __builtin_amdgcn_raw_buffer_load_b128(wr, wlane + h * 1024, wofs, 0));
    wofs += 2048;
  };
#pragma unroll
  for (int i = 0; i < D; ++i) wload(i);
  // The reduce launch of a layer whose K is split makes a NaN 0 (fmaxf), the unsplit kernels' ReLU
  // keeps a positive one.  A NaN of the matrix cores is negative, so a positive one comes from
  // the layer's scale or shift: turned here, once, relu_b does for both.
  constexpr int kFirstA = (HASB ? MID : 0) + 4 * MID;
  const bool split_b = HASB && a.b_per < 9 * MID / 64, split_a = HASA && a.a_per < 4 * MID / 64;
  for (int i = tid; i < TAB; i += NW * 64) {
    const bool split = i < MID ? split_b : (i >= kFirstA && split_a);
    const float sc = a.table[2 * i], sh = a.table[2 * i + 1];
    tab[2 * i] = split ? negative_nan(sc) : sc;
    tab[2 * i + 1] = split ? negative_nan(sh) : sh;
  }
  if (tid < 8) zero[tid] = make_uint4(0u, 0u, 0u, 0u);
  uint4* const in0 = HASB ? xbuf : mid;
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int it = i * (NW * 64) + tid;
    if (it < IN_ROWS * NCH) in0[it] = pv[i];
  }
  lds_barrier();

  const char* const ldsb = (const char*)lds;
  auto rd = [&](int byte) { return *(const bf16x8_b*)(ldsb + byte); };
  constexpr int MIDB = XROWS * NCH * 16, ZEROB = MIDB + BM * NCH * 16;

  f32x16_b acc[TP];
  auto clear = [](f32x16_b (&v)[TP]) {
#pragma unroll
    for (int t = 0; t < TP; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) v[t][e] = 0.f;
  };
  // partial sums of K are kept apart and added in order, as the split-K launches add them
  auto fold = [](f32x16_b (&sum)[TP], f32x16_b (&part)[TP]) {
#pragma unroll
    for (int t = 0; t < TP; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sum[t][e] += part[t][e];
        part[t][e] = 0.f;
      }
  };
  auto mfma_step = [&](f32x16_b (&c)[TP], bf16x8_b (&w)[2], bf16x8_b (&x)[TP][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < TP; ++t)
        c[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[h], x[t][h], c[t], 0, 0, 0);
  };
  // scale and shift of this lane's 4 channels of group g in the table rows from `base`
  // ([scale, shift] pairs), applied as the layer kernels do
  auto folded = [&](const f32x16_b& v, int g, int base, float (&o)[4]) {
    const float4 p = *(const float4*)(tab + 2 * (base + 8 * g + 4 * fk));
    const float4 s = *(const float4*)(tab + 2 * (base + 8 * g + 4 * fk) + 4);
    o[0] = v[4 * g + 0] * p.x + p.y;
    o[1] = v[4 * g + 1] * p.z + p.w;
    o[2] = v[4 * g + 2] * s.x + s.y;
    o[3] = v[4 * g + 3] * s.z + s.w;
  };

  bf16x8_b xf[2][TP][2];
  if constexpr (HASB) {
    // ---- 3x3: K ordered (channel block of 64, tap, channel)
    int prow[TP];
    unsigned ok[TP];   // bit t: tap t of this lane's pixel lies inside the image
#pragma unroll
    for (int t = 0; t < TP; ++t) {
      const int m = m0 + t * 32 + frow;
      const int w = m % a.W, h = (m / a.W) % a.H;
      unsigned v = 0;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int hh = h + k / 3 - 1, ww = w + k % 3 - 1;
        if (m < a.M && (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W) v |= 1u << k;
      }
      ok[t] = v;
      prow[t] = t * 32 + frow;   // patch row of tap (0, 0) is the pixel's own index
    }
    int tap = 0, tv = 0, toff = 0, cb = 0;   // the tap of the step being read: index, column, row offset, block
    int ad[TP];
    auto address = [&]() {
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        const int r = prow[t] + toff;
        const int at = r * (NCH * 16) + ((((cb * 8) ^ rsw<MID>(r)) ^ fk) << 4);
        ad[t] = (ok[t] >> tap) & 1u ? at : ZEROB + (fk << 4);
      }
      if (++tap == 9) {
        tap = 0; tv = 0; toff = 0;
        if (++cb == MID / 64) cb = 0;   // after the last tap: a read that is not used
      } else if (++tv == 3) {
        tv = 0;
        toff += a.W - 2;
      } else {
        ++toff;
      }
    };
    auto frags = [&](bf16x8_b (&x)[TP][2], int half) {
#pragma unroll
      for (int t = 0; t < TP; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) x[t][h] = rd(ad[t] ^ ((half * 4 + h * 2) << 4));
    };
    f32x16_b tot[TP];
    clear(acc);
    clear(tot);
    address();
    frags(xf[0], 0);
    int left = a.b_per;   // K tiles of 64 left in this partial sum
    for (int g = 0; g < NB / D; ++g) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        if (i & 1) {
          address();
          frags(xf[0], 0);
        } else {
          frags(xf[1], 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        mfma_step(acc, wf[i], xf[i & 1]);
        __builtin_amdgcn_sched_barrier(0);
        wload(i);
        if ((i & 1) && --left == 0) {
          fold(tot, acc);
          left = a.b_per;
        }
      }
    }
    if (left != a.b_per) fold(tot, acc);
    // the rounded 3x3 output into LDS
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        float o[4];
        folded(tot[t], g, wave * 32, o);
        const int r = t * 32 + frow;
        uint2 p;
        p.x = pack2_b(relu_b(o[0]), relu_b(o[1]));
        p.y = pack2_b(relu_b(o[2]), relu_b(o[3]));
        *((uint2*)(mid + r * NCH + ((4 * wave + g) ^ rsw<MID>(r))) + fk) = p;
      }
    lds_barrier();
  }

  // ---- expansion in chunks of MID channels, each a K slice of the next reduction
  constexpr int CTAB = HASB ? MID : 0, ATAB = CTAB + 4 * MID;
  const int rpl = lane >> 2, roct = lane & 3;   // 16-byte accesses: 16 pixels x 4 octets of the wave's channels
  int cad[TP];   // LDS byte of this lane's first chunk in a row-major tile of BM rows
#pragma unroll
  for (int t = 0; t < TP; ++t) {
    const int r = t * 32 + frow;
    cad[t] = r * (NCH * 16) + ((rsw<MID>(r) ^ fk) << 4);
  }
  f32x16_b acc2[TP], tot2[TP];
  clear(acc2);
  clear(tot2);
  int left2 = a.a_per;
  auto step_frags = [&](bf16x8_b (&x)[TP][2], int base, int s) {
#pragma unroll
    for (int t = 0; t < TP; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) x[t][h] = rd(base + (cad[t] ^ ((s * 4 + h * 2) << 4)));
  };
  for (int c = 0; c < 4; ++c) {
    const int ch = c * MID + wave * 32;   // this wave's channels of the chunk
    uint4 rv[BM / 16];
#pragma unroll
    for (int p = 0; p < BM / 16; ++p) {
      const int m = m0 + p * 16 + rpl;
      const unsigned off = m < a.M ? ((unsigned)m * (4 * MID) + ch + 8 * roct) * 2u : 0xFFFFFFF0u;
      rv[p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rr, (int)off, 0, 0));
    }
    clear(acc);
    step_frags(xf[0], MIDB, 0);
#pragma unroll
    for (int i = 0; i < D; ++i) {
      if (i + 1 < D) step_frags(xf[(i + 1) & 1], MIDB, i + 1);
      __builtin_amdgcn_sched_barrier(0);
      mfma_step(acc, wf[i], xf[i & 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (HASA || c < 3) wload(i);
    }
    // every wave has read the previous chunk (the patch before it: at the 3x3's barrier)
    if (HASA && c > 0) lds_barrier();
    // the wave's residual slice, then its outputs in place of it
#pragma unroll
    for (int p = 0; p < BM / 16; ++p) {
      const int r = p * 16 + rpl;
      xbuf[r * NCH + ((4 * wave + roct) ^ rsw<MID>(r))] = rv[p];
    }
    lds_wave_sync();
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        const int r = t * 32 + frow;
        uint2* at = (uint2*)(xbuf + r * NCH + ((4 * wave + g) ^ rsw<MID>(r))) + fk;
        const uint2 res = *at;
        float o[4];
        folded(acc[t], g, CTAB + ch, o);
        o[0] += bf2f_b(res.x & 0xFFFFu);
        o[1] += bf2f_b(res.x >> 16);
        o[2] += bf2f_b(res.y & 0xFFFFu);
        o[3] += bf2f_b(res.y >> 16);
        uint2 pk;
        pk.x = pack2_b(relu_b(o[0]), relu_b(o[1]));
        pk.y = pack2_b(relu_b(o[2]), relu_b(o[3]));
        *at = pk;
      }
    if (HASA) lds_barrier();
    else lds_wave_sync();
#pragma unroll
    for (int p = 0; p < BM / 16; ++p) {
      const int r = p * 16 + rpl, m = m0 + r;
      if (m < a.M)
        *(uint4*)((bf16_t*)a.y + (size_t)m * (4 * MID) + ch + 8 * roct) =
            xbuf[r * NCH + ((4 * wave + roct) ^ rsw<MID>(r))];
    }
    if constexpr (HASA) {
      step_frags(xf[0], 0, 0);
#pragma unroll
      for (int i = 0; i < D; ++i) {
        if (i + 1 < D) step_frags(xf[(i + 1) & 1], 0, i + 1);
        __builtin_amdgcn_sched_barrier(0);
        mfma_step(acc2, wf[i], xf[i & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (c < 3) wload(i);
        if ((i & 1) && --left2 == 0) {
          fold(tot2, acc2);
          left2 = a.a_per;
        }
      }
    } else {
      lds_wave_sync();   // the slice has been read before the next chunk rewrites it
    }
  }
  if constexpr (HASA) {
    if (left2 != a.a_per) fold(tot2, acc2);
    // every wave is past the last expansion's reads of `mid`
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int t = 0; t < TP; ++t) {
        float o[4];
        folded(tot2[t], g, ATAB + wave * 32, o);
        const int r = t * 32 + frow;
        uint2 p;
        p.x = pack2_b(relu_b(o[0]), relu_b(o[1]));
        p.y = pack2_b(relu_b(o[2]), relu_b(o[3]));
        *((uint2*)(mid + r * NCH + ((4 * wave + g) ^ rsw<MID>(r))) + fk) = p;
      }
    lds_wave_sync();
#pragma unroll
    for (int p = 0; p < BM / 16; ++p) {
      const int r = p * 16 + rpl, m = m0 + r;
      if (m < a.M)
        *(uint4*)((bf16_t*)a.z + (size_t)m * MID + wave * 32 + 8 * roct) =
            mid[r * NCH + ((4 * wave + roct) ^ rsw<MID>(r))];
    }
  }
}

// The block's weights in the order in which wave w of block_kernel reads them: the steps
// of the 3x3 (9 MID / 32, or none), then per chunk c of the expansion its MID / 32 steps
// and those of the reduction's K slice c; a step is two fragments (16 terms each) of 64
// lanes x 8 terms, lane fk * 32 + r holding row r, terms 8 fk .. 8 fk + 7.  One thread per
// lane of a fragment.
__global__ void pack_block_weights_kernel(const bf16_t* wb, int kpb, const bf16_t* wc, int kpc, const bf16_t* wa,
                                          int kpa, int mid, bf16_t* out, long long total) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int D = mid / 32, nb = wb ? 9 * D : 0, per_chunk = wa ? 2 * D : D, steps = nb + 4 * per_chunk;
  const int lane = (int)(idx & 63), h = (int)(idx >> 6) & 1;
  const long long ws = idx >> 7;
  const int w = (int)(ws / steps), s = (int)(ws - (long long)w * steps);
  const int row = w * 32 + (lane & 31), k0 = h * 16 + 8 * (lane >> 5);
  const bf16_t* src;
  if (s < nb) {
    src = wb + (size_t)row * kpb + s * 32 + k0;
  } else {
    const int c = (s - nb) / per_chunk, t = (s - nb) - c * per_chunk;
    if (t < D) src = wc + (size_t)(c * mid + row) * kpc + t * 32 + k0;
    else src = wa + (size_t)row * kpa + (c * D + t - D) * 32 + k0;
  }
  *(uint4*)(out + idx * 8) = *(const uint4*)src;
}

size_t block_weight_bytes(int mid, bool has_b, bool has_a) {
  const int D = mid / 32;
  return (size_t)(mid / 32) * ((has_b ? 9 * D : 0) + 4 * (has_a ? 2 * D : D)) * 2048;
}

hipError_t launch_pack_block_weights(const bf16_t* wb, int kpb, const bf16_t* wc, int kpc, const bf16_t* wa, int kpa,
                                     int mid, bf16_t* out, hipStream_t s) {
  const long long total = (long long)block_weight_bytes(mid, wb != nullptr, wa != nullptr) / 16;
  launch(pack_block_weights_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), s, wb, kpb, wc, kpc, wa, kpa,
         mid, out, total);
  return hipGetLastError();
}

#define RAFIKI_BLOCKS(X) \
  X(64, 64, true, true) X(64, 64, true, false) X(64, 64, false, true)       \
  X(64, 32, true, true) X(64, 32, true, false) X(64, 32, false, true)       \
  X(128, 64, true, true) X(128, 64, true, false) X(128, 64, false, true)    \
  X(128, 32, true, true) X(128, 32, true, false) X(128, 32, false, true)    \
  X(256, 64, true, true) X(256, 64, true, false) X(256, 64, false, true)    \
  X(256, 32, true, true) X(256, 32, true, false) X(256, 32, false, true)
#define RAFIKI_INST(MID, BM, HB, HA) template __global__ void block_kernel<MID, BM, HB, HA>(BlockArgs);
RAFIKI_BLOCKS(RAFIKI_INST)
#undef RAFIKI_INST

hipError_t launch_block(const BlockArgs& a, int mid, int bm, hipStream_t s) {
  const bool hb = a.has_b != 0, ha = a.z != nullptr;
  const dim3 grid((unsigned)((a.M + bm - 1) / bm));
#define RAFIKI_CASE(MID, BM, HB, HA)                                        \
  if (mid == MID && bm == BM && hb == HB && ha == HA) {                     \
    launch((block_kernel<MID, BM, HB, HA>), grid, dim3(MID * 2), s, a);     \
    return hipGetLastError();                                               \
  }
  RAFIKI_BLOCKS(RAFIKI_CASE)
#undef RAFIKI_CASE
  return hipErrorInvalidValue;
}
#undef RAFIKI_BLOCKS

}  // namespace rafiki
