// fp32 image CNNs of a few small layers, by runs of layers in one launch (gfx950).
//
// The two toy CNNs of eight 32 x 32 images were seven launches of 4 to 7 us for 52 MFLOP:
// every layer paid a launch, one latency to fetch what the last had stored, and a grid too
// small to hide it.  Two kernels replace six of the launches.
//
// chain_f32_kernel runs the leading run of convolutions and 2x2 max-pools of one model over a
// band of output rows of one image, straight from the NCHW request: each layer's rows for the
// band (and the halo the next layer needs) are computed into LDS, zero rows and columns
// standing for the padding, and only the last layer's band is stored.  The weights of every
// layer come to LDS with the image, so one latency covers both.  Convolutions run on the fp32
// matrix cores in 16 pixel x 16 channel tiles (v_mfma_f32_16x16x4_f32: four input channels of
// one tap), whose operands are one LDS word per lane each; as FMAs with the weights in scalar
// registers the same kernel waited for scalar loads (26 us against 13 for the two toy
// CNNs at eight images).  Bands recompute their halo (a third of the first layer at four rows
// of sixteen) for four times the compute units.
//
// tail_f32_kernel takes the mean over positions and the final FC of one request.
//
// Sums are fp32 throughout, in (tap, channel) order with four channels per instruction;
// padding adds exact zero products.
#include "kernels.h"

namespace rafiki {

namespace {
typedef float f32x4_c __attribute__((ext_vector_type(4)));

// One 16 x 16 tile of a convolution layer: pixels px0 .. + 15 (row-major in the band) by
// channels co0 .. + 15.  Lane (i, k) = (lane % 16, lane / 16) feeds pixel i and channel i at input
// channel 4 c4 + k; it ends with channels co0 + 4 k .. + 3 of pixel i.  KS: kernel size; C4: input
// channels / 4 (0: L.C4).
template <int KS, int C4>
__device__ __forceinline__ void chain_conv(const ChainLayer& L, const float* lds, float* y, const float* fold, int px0,
                                           int co0, int row0, bool last, int n, int lane) {
  const int i = lane & 15, k = lane >> 4;
  const int px = px0 + i, r = px / L.Wo, c = px - r * L.Wo;
  const bool live = px < L.rows * L.Wo;
  const float* xp = lds + L.in_off + (live ? r * L.in_stride + c : 0) + k * L.in_plane;   // tap (0, 0)
  const float* wp = lds + L.w_off + k * L.ldc + co0 + i;
  f32x4_c acc = {0.f, 0.f, 0.f, 0.f};
  const int c4n = C4 ? C4 : L.C4;
#pragma unroll
  for (int u = 0; u < KS; ++u)
#pragma unroll
    for (int v = 0; v < KS; ++v) {
      const float* xt = xp + u * L.in_stride + v;
      const float* wt = wp + (u * KS + v) * c4n * 4 * L.ldc;
#pragma unroll 4
      for (int q = 0; q < c4n; ++q)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[q * 4 * L.ldc], xt[q * 4 * L.in_plane], acc, 0, 0, 0);
    }
  const int ho = row0 + r, co = co0 + 4 * k;
  const bool inside = live && (unsigned)ho < (unsigned)L.Ho;
  float o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    o[j] = acc[j] * fold[2 * (co + j)] + fold[2 * (co + j) + 1];
    if (L.relu) o[j] = fmaxf(o[j], 0.f);
  }
  if (last) {
    if (inside && co < L.ldy)
      *(float4*)(y + (((size_t)n * L.Ho + ho) * L.Wo + c) * L.ldy + co) = make_float4(o[0], o[1], o[2], o[3]);
    return;
  }
  if (!live) return;
  float* out = (float*)lds + L.out_off + r * L.out_stride + c;
#pragma unroll
  for (int j = 0; j < 4; ++j)   // rows outside the image are the next layer's padding
    if (co + j < L.Co) out[(co + j) * L.out_plane] = inside ? o[j] : 0.f;
}
}  // namespace

__global__ __launch_bounds__(kChainThreads) void chain_f32_kernel(ChainArgs a) {
  extern __shared__ float chain_lds[];
  const int n = blockIdx.x, band = blockIdx.y, mem = blockIdx.z, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = kChainThreads / 64;
  // Everything the band reads from memory is requested before anything is waited for: first
  // the image's words, U per thread and round, then the weights and folds of every layer.
  constexpr int U = 4;
  const int in_row0 = band * a.band_step[0] + a.band_base[0];
  const int per = a.in_rows * a.W, words = a.C * per;
  float img[U];
  int at[U];
  auto fetch = [&](int base) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = base + k * kChainThreads + tid;
      const int c = i / per, p = i - c * per, r = p / a.W, w = p - r * a.W, h = in_row0 + r;
      const bool ok = i < words && (unsigned)h < (unsigned)a.H;
      at[k] = ok ? c * a.in_plane + r * a.in_stride + a.in_col + w : -1;
      img[k] = ok ? a.x[((size_t)(n * a.C + c) * a.H + h) * a.W + w] : 0.f;
    }
  };
  auto put = [&]() {
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (at[k] >= 0) chain_lds[at[k]] = img[k];
  };
  fetch(0);
  for (int l = 0; l < a.n_layers; ++l) {
    const ChainLayer& L = a.layer[l];
    if (L.k == 0) continue;
    const float* w = a.w[mem][l];
    const int quads = L.ldc / 4, rows = L.C4 * 4, total = L.k * L.k * rows * quads;
    for (int base = 0; base < total; base += U * kChainThreads) {
      float4 v[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int i = base + k * kChainThreads + tid;
        const int row = i / quads, q = i - row * quads, tap = row / rows, ci = row - tap * rows;
        v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < total && ci < L.C) v[k] = *(const float4*)(w + (size_t)(tap * L.Cs + ci) * L.Co_pad + 4 * q);   // ldc <= Co_pad
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int i = base + k * kChainThreads + tid;
        if (i < total) *(float4*)(chain_lds + L.w_off + 4 * i) = v[k];
      }
    }
    for (int i = tid; i < L.ldc; i += kChainThreads) {
      const float sc = a.scale[mem][l][i], sh = a.shift[mem][l][i];
      chain_lds[L.fold_off + 2 * i] = sc;
      chain_lds[L.fold_off + 2 * i + 1] = sh;
    }
  }
  // the band's rows of the request in zeroed buffers (disjoint from the weights)
  for (int i = tid; i < a.act_floats / 4; i += kChainThreads) ((float4*)chain_lds)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  put();
  for (int base = U * kChainThreads; base < words; base += U * kChainThreads) {
    fetch(base);
    put();
  }
  __syncthreads();
  for (int l = 0; l < a.n_layers; ++l) {
    const ChainLayer& L = a.layer[l];
    const int row0 = band * a.band_step[l + 1] + a.band_base[l + 1];
    const bool last = l == a.n_layers - 1;
    float* y = a.y[mem];
    if (L.k == 0) {   // 2x2 stride-2 max-pool
      const float* in = chain_lds + L.in_off;
      float* out = chain_lds + L.out_off;
      const int px = L.rows * L.Wo;
      for (int i = tid; i < (last ? L.ldy : L.Co) * px; i += kChainThreads) {
        const int c = i / px, p = i - c * px, r = p / L.Wo, w = p - r * L.Wo;
        const float* q = in + (c < L.Co ? c : 0) * L.in_plane + 2 * r * L.in_stride + 2 * w;
        const float m = c >= L.Co ? 0.f :   // storage padding of the stored rows
            fmaxf(fmaxf(q[0], q[1]), fmaxf(q[L.in_stride], q[L.in_stride + 1]));
        const bool inside = (unsigned)(row0 + r) < (unsigned)L.Ho;
        if (!last) out[c * L.out_plane + r * L.out_stride + w] = inside ? m : 0.f;
        else if (inside) y[(((size_t)n * L.Ho + row0 + r) * L.Wo + w) * L.ldy + c] = m;
      }
    } else {
      const int blocks = (L.rows * L.Wo + 15) / 16, tasks = blocks * (L.ldc / 16);
      const float* fold = chain_lds + L.fold_off;
      for (int t = wave; t < tasks; t += NW) {
        const int px0 = t % blocks * 16, co0 = t / blocks * 16;
        if (L.k == 1) chain_conv<1, 0>(L, chain_lds, y, fold, px0, co0, row0, last, n, lane);
        else if (L.C4 == 1) chain_conv<3, 1>(L, chain_lds, y, fold, px0, co0, row0, last, n, lane);
        else chain_conv<3, 0>(L, chain_lds, y, fold, px0, co0, row0, last, n, lane);
      }
    }
    __syncthreads();
  }
}

hipError_t launch_chain_f32(const ChainArgs& a, int n, int bands, int members, hipStream_t s) {
  if (n < 1 || bands < 1 || members < 1 || members > kMaxGroup || a.n_layers < 1 || a.n_layers > kChainMaxLayers ||
      a.lds_floats * 4 > kChainLdsBytes)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)n, (unsigned)bands, (unsigned)members), block(kChainThreads);
  const size_t lds = (size_t)a.lds_floats * 4;
  const LaunchEvents& ev = launch_events();
  if (ev.start || ev.stop) hipExtLaunchKernelGGL(chain_f32_kernel, grid, block, lds, s, ev.start, ev.stop, 0, a);
  else hipLaunchKernelGGL(chain_f32_kernel, grid, block, lds, s, a);
  return hipGetLastError();
}

// Mean over HW positions of [HW][Cs], then z = scale (W x) + shift: one workgroup per request
// and member.  Thread (slice, channel) sums every S-th position, S = 256 / Cs slices, which are
// then added in order; output j sums its products in channel order.
__global__ __launch_bounds__(256) void tail_f32_kernel(TailArgs a) {
  __shared__ float part[256];
  __shared__ float mean[256];
  const int n = blockIdx.x, mem = blockIdx.y, t = threadIdx.x;
  const int S = 256 / a.Cs, sl = t / a.Cs, c = t - sl * a.Cs;
  const float* x = a.x[mem] + (size_t)n * a.HW * a.Cs;
  float acc = 0.f;
  if (sl < S) {
#pragma unroll 8
    for (int p = sl; p < a.HW; p += S) acc += x[(size_t)p * a.Cs + c];
  }
  part[t] = acc;
  __syncthreads();
  if (t < a.Cs) {
    for (int k = 1; k < S; ++k) acc += part[k * a.Cs + t];
    mean[t] = acc * (1.0f / (float)a.HW);
  }
  __syncthreads();
  for (int j = t; j < a.n_out; j += 256) {
    const float* w = a.w[mem] + j;
    float z = 0.f;
#pragma unroll 8
    for (int k = 0; k < a.Cs; ++k) z = fmaf(mean[k], w[(size_t)k * a.Co_pad], z);
    z = z * a.scale[mem][j] + a.shift[mem][j];
    a.y[mem][(size_t)n * a.ldy + j] = a.relu ? fmaxf(z, 0.f) : z;
  }
}

hipError_t launch_tail_f32(const TailArgs& a, int n, int members, hipStream_t s) {
  if (n < 1 || members < 1 || members > kMaxGroup || a.Cs < 1 || a.Cs > 256 || a.HW < 1) return hipErrorInvalidValue;
  launch(tail_f32_kernel, dim3((unsigned)n, (unsigned)members), dim3(256), s, a);
  return hipGetLastError();
}

}  // namespace rafiki
