// Fused conv1d branches over a token sequence, from a table of per-tap products (gfx950).
//
// A convolution over embedded tokens is linear in each token's embedding, so its sum over
// the kernel's taps is a sum of rows of a table that depends on the weights alone:
//   T[id][(branch, tap, filter)] = sum_c E[id][c] * W_branch[filter][c][tap]   (fp32)
// built once with the weights.  A request then adds, at each position, one table value per
// tap instead of one product per tap and embedding channel: for 300 channels 4 bytes
// fetched stand in for 600 FLOPs.  The kernel is bound by fetching rows at random
// positions of the table (4.8 KB a token for kernels of 3, 4 and 5 taps x 100 filters).
//
// One workgroup takes one request (or a slice of its positions) of one model.  Thread
// (segment, quad) keeps the running maximum of 4 neighbouring filters of one branch over
// its segment of positions, so the quads of a row are adjacent 16-byte loads and every
// byte of the row is used once; the segments meet in LDS.  Each position applies the folded
// scale and shift (a batch-norm scale may be negative) before the maximum; rounding to bf16
// is monotone, so one rounding after the maximum equals the maximum of rounded values.
#include "kernels.h"

namespace rafiki {

namespace {
__device__ __forceinline__ uint32_t f2bf_t(float f) {   // nearest, ties to even (finite)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}
}  // namespace

// KW: the most taps of any branch.
template <int KW>
__global__ __launch_bounds__(kTapThreads) void tap_table_kernel(TapArgs a) {
  extern __shared__ uint4 tap_lds[];
  unsigned* const row = (unsigned*)tap_lds;                            // byte offset of each token's row
  float4* const red = (float4*)(row + ((a.len + KW + 3) & ~3));        // [segments][quads]
  const int n = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
  const float* T = a.table[0];
  const float* scale = a.scale[0];
  const float* shift = a.shift[0];
  bf16_t* y = a.y[0];
  unsigned* slot = a.slot[0];
#pragma unroll
  for (int k = 1; k < kMaxGroup; ++k)
    if (blockIdx.z == (unsigned)k) {
      T = a.table[k]; scale = a.scale[k]; shift = a.shift[k]; y = a.y[k]; slot = a.slot[k];
    }
  // positions [pa, pb) of this part; the last taps reach KW - 1 tokens further
  const int pa = part * a.part_len, pb = min(pa + a.part_len, a.len);
  const int ntok = min(pb + KW - 1, a.len) - pa;
  for (int i = tid; i < ntok; i += blockDim.x) {
    const int id = a.tok[(long long)n * a.len + pa + i];
    row[i] = (unsigned)((unsigned)id < (unsigned)a.vocab ? id : a.vocab) * (unsigned)(a.ldt * 4);   // row vocab: zeros
  }
  __syncthreads();
  const int seg = tid / a.quads, quad = tid - seg * a.quads;
  // the quad's branch: taps, positions, first float of tap 0, floats per tap, output row
  int kw = 0, base = 0, step = 0, out = 0, left = 0;
#pragma unroll
  for (int i = 0; i < kMaxReduceSegs; ++i)
    if (i < a.n_branches && quad >= a.quad0[i]) {
      kw = a.kw[i];
      step = 4 * ((a.cnt[i] + 3) / 4);
      base = a.first[i] + 4 * (quad - a.quad0[i]);
      out = a.row[i] + 4 * (quad - a.quad0[i]);
      left = a.cnt[i] - 4 * (quad - a.quad0[i]);
    }
  float4 m = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
  if (seg < a.segments) {
    float sc[4], sh[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sc[j] = j < left ? scale[out + j] : 0.f;
      sh[j] = j < left ? shift[out + j] : 0.f;
    }
    const int per = (pb - pa + a.segments - 1) / a.segments;
    const int p0 = pa + seg * per, p1 = min(min(p0 + per, pb), a.len - kw + 1);
    const char* const Tb = (const char*)(T + base);
    constexpr int U = KW <= 4 ? 4 : (KW <= 6 ? 3 : 2);   // positions in flight
    for (int p = p0; p < p1; p += U) {
      float4 v[U][KW];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = min(p + u, p1 - 1) - pa;
#pragma unroll
        for (int t = 0; t < KW; ++t)
          if (t < kw) v[u][t] = *(const float4*)(Tb + row[q + t] + (size_t)(t * step * 4));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float4 s = v[u][0];
#pragma unroll
        for (int t = 1; t < KW; ++t)
          if (t < kw) { s.x += v[u][t].x; s.y += v[u][t].y; s.z += v[u][t].z; s.w += v[u][t].w; }
        m.x = fmaxf(m.x, s.x * sc[0] + sh[0]);
        m.y = fmaxf(m.y, s.y * sc[1] + sh[1]);
        m.z = fmaxf(m.z, s.z * sc[2] + sh[2]);
        m.w = fmaxf(m.w, s.w * sc[3] + sh[3]);
      }
    }
    red[seg * a.quads + quad] = m;
  }
  __syncthreads();
  if (seg == 0) {
    for (int s = 1; s < a.segments; ++s) {
      const float4 o = red[s * a.quads + quad];
      m.x = fmaxf(m.x, o.x); m.y = fmaxf(m.y, o.y); m.z = fmaxf(m.z, o.z); m.w = fmaxf(m.w, o.w);
    }
    const float v[4] = {m.x, m.y, m.z, m.w};
    int dst = 0;
#pragma unroll
    for (int i = 0; i < kMaxReduceSegs; ++i)
      if (i < a.n_branches && quad >= a.quad0[i]) dst = a.dst[i] + 4 * (quad - a.quad0[i]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j >= left) break;
      const uint32_t r = f2bf_t(a.relu ? fmaxf(v[j], 0.f) : v[j]);
      if (gridDim.y == 1) y[(long long)n * a.ldy + dst + j] = (bf16_t)r;
      else if (v[j] > -INFINITY) atomicMax(slot + (long long)n * a.ldslot + out + j, max_key(__uint_as_float(r << 16)));
    }
  }
  if (gridDim.y == 1)
    for (int c = a.zero_from + tid; c < a.ldy; c += blockDim.x) y[(long long)n * a.ldy + c] = 0;
}

hipError_t launch_tap_table(const TapArgs& a0, int n, int parts, hipStream_t s) {
  TapArgs a = a0;
  if (n < 1 || parts < 1 || a.n_members < 1 || a.n_members > kMaxGroup || a.n_branches < 1 ||
      a.n_branches > kMaxReduceSegs || a.quads < 1 || a.quads > kTapThreads || a.len < 1 || a.len > kTapMaxLen)
    return hipErrorInvalidValue;
  int kw = 1;
  for (int i = 0; i < a.n_branches; ++i) kw = a.kw[i] > kw ? a.kw[i] : kw;
  a.part_len = (a.len + parts - 1) / parts;
  a.segments = kTapThreads / a.quads;
  if (a.segments > 8) a.segments = 8;
  const int threads = (a.segments * a.quads + 63) / 64 * 64;
  const size_t lds = (size_t)((a.len + 8 + 3) & ~3) * 4 + 16 + (size_t)a.segments * a.quads * 16;
  const dim3 grid((unsigned)n, (unsigned)parts, (unsigned)a.n_members);
#define RAFIKI_TAP(K)                                                                      \
  case K:                                                                                  \
    if (launch_events().start || launch_events().stop)                                     \
      hipExtLaunchKernelGGL((tap_table_kernel<K>), grid, dim3(threads), lds, s, launch_events().start, \
                            launch_events().stop, 0, a);                                   \
    else                                                                                   \
      hipLaunchKernelGGL((tap_table_kernel<K>), grid, dim3(threads), lds, s, a);           \
    break;
  switch (kw) {
    RAFIKI_TAP(1) RAFIKI_TAP(2) RAFIKI_TAP(3) RAFIKI_TAP(4) RAFIKI_TAP(5) RAFIKI_TAP(6) RAFIKI_TAP(7) RAFIKI_TAP(8)
    default: return hipErrorInvalidValue;
  }
#undef RAFIKI_TAP
  return hipGetLastError();
}

}  // namespace rafiki
