// Token embedding with the first RMSNorm and the rotary factors, and RMSNorm.
//
// RMSNorm: h = bf16(x * (mean(x^2) + eps)^(-1/2) * g) with x the float32
// residual row; one workgroup per row, float4 loads, a wave64 butterfly sum
// and a cross-wave sum through LDS.  Rows up to 8192 wide are held in
// registers between the two passes.
#include "common.h"
#include "kernels.h"

namespace pallas {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float block_sum(float v, float* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < kThreads / 64; ++i) t += sh[i];
  return t;
}

// Writes h[i..i+3] = bf16(x * inv * g)
__device__ __forceinline__ void store_norm4(uint16_t* h, const uint16_t* g, int i, f32x4 x, float inv) {
  const u32x2 gg = *reinterpret_cast<const u32x2*>(g + i);
  u32x2 out;
  out.x = pack_bf2(x.x * inv * bflo(gg.x), x.y * inv * bfhi(gg.x));
  out.y = pack_bf2(x.z * inv * bflo(gg.y), x.w * inv * bfhi(gg.y));
  *reinterpret_cast<u32x2*>(h + i) = out;
}

// The start of a call, one workgroup per row: the row's embedding as its
// residual, the first RMSNorm, the row's rotary factors (tab[row][i] = (cos,
// sin)(pos theta^(-2i/d)), in double), clears of the counters a decode step
// needs, and its rows' shared-slot flags.  One launch instead of three of 3 to 5 us.
__global__ __launch_bounds__(kThreads) void embed_rmsnorm_kernel(
    const int32_t* __restrict__ ids, const uint16_t* __restrict__ E, const uint16_t* __restrict__ g,
    float* __restrict__ r, uint16_t* __restrict__ h, int H, float eps, int vocab, int32_t* err, RowMap rm, int half,
    double log2_theta_over_half, float* __restrict__ tab, ClearSpan ca, ClearSpan cb, SharedSlots sl) {
  __shared__ float sh[kThreads / 64];
  __shared__ int wpage[kMaxSeqs];
  const int t = blockIdx.x;
  for (int i = t * kThreads + threadIdx.x; i < ca.n + cb.n; i += gridDim.x * kThreads) {
    if (i < ca.n) ca.p[i] = 0;
    else cb.p[i - ca.n] = 0;
  }
  if (sl.flag) {
    // Does a page that some row writes hold a position before this row's own?
    if (threadIdx.x < rm.n_seqs)
      wpage[threadIdx.x] = sl.bt[static_cast<int64_t>(threadIdx.x) * sl.max_pages + rm.base_pos[threadIdx.x] / sl.page];
    __syncthreads();
    const int n = rm.base_pos[t];
    int any = 0;
    for (int e = threadIdx.x; e * sl.page < n; e += kThreads) {
      const int pg = sl.bt[static_cast<int64_t>(t) * sl.max_pages + e];
      if (pg < 0 || pg >= sl.num_pages) continue;
      for (int i = 0; i < rm.n_seqs; ++i) any |= wpage[i] == pg && e * sl.page + rm.base_pos[i] % sl.page < n;
    }
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) sl.flag[t] = any;
  }
  if (threadIdx.x < half) {
    const int s = row_seq(rm, t);
    const double pos = double(rm.base_pos[s] + (t - rm.cu[s]));
    // theta^(-2i/d) = 2^(-i * log2(theta) / (d/2))
    const double inv_freq = exp2(-double(threadIdx.x) * log2_theta_over_half);
    double sn, cs;
    sincos(pos * inv_freq, &sn, &cs);
    float* dst = tab + 2 * (static_cast<int64_t>(t) * half + threadIdx.x);
    dst[0] = static_cast<float>(cs);
    dst[1] = static_cast<float>(sn);
  }
  int id = ids[t];
  if (id < 0 || id >= vocab) {
    if (threadIdx.x == 0 && err) atomicOr(err, static_cast<int32_t>(PALLAS_DEVERR_TOKEN));
    id = 0;
  }
  const uint16_t* e = E + static_cast<int64_t>(id) * H;
  float* rr = r + static_cast<int64_t>(t) * H;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < H; i += kThreads * 4) {
    const u32x2 w = *reinterpret_cast<const u32x2*>(e + i);
    const f32x4 x = {bflo(w.x), bfhi(w.x), bflo(w.y), bfhi(w.y)};
    *reinterpret_cast<f32x4*>(rr + i) = x;
    ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
  }
  const float inv = rsqrtf(block_sum(ss, sh) / H + eps);
  uint16_t* hh = h + static_cast<int64_t>(t) * H;
  for (int i = threadIdx.x * 4; i < H; i += kThreads * 4) {
    const u32x2 w = *reinterpret_cast<const u32x2*>(e + i);
    const f32x4 x = {bflo(w.x), bfhi(w.x), bflo(w.y), bfhi(w.y)};
    store_norm4(hh, g, i, x, inv);
  }
}

// Rows of up to kRegVecs * kThreads * 4 elements stay in registers between
// the sum of squares and the scaling, so a row is read from memory once.
constexpr int kRegVecs = 8;

__global__ __launch_bounds__(kThreads) void rmsnorm_reg_kernel(const float* __restrict__ r,
                                                               const uint16_t* __restrict__ g,
                                                               uint16_t* __restrict__ h, int H,
                                                               float eps) {
  __shared__ float sh[kThreads / 64];
  const int t = blockIdx.x;
  const float* rr = r + static_cast<int64_t>(t) * H;
  f32x4 x[kRegVecs];
  float ss = 0.f;
#pragma unroll
  for (int v = 0; v < kRegVecs; ++v) {
    const int i = (v * kThreads + threadIdx.x) * 4;
    x[v] = i < H ? *reinterpret_cast<const f32x4*>(rr + i) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int v = 0; v < kRegVecs; ++v) ss += x[v].x * x[v].x + x[v].y * x[v].y + x[v].z * x[v].z + x[v].w * x[v].w;
  const float inv = rsqrtf(block_sum(ss, sh) / H + eps);
  uint16_t* hh = h + static_cast<int64_t>(t) * H;
#pragma unroll
  for (int v = 0; v < kRegVecs; ++v) {
    const int i = (v * kThreads + threadIdx.x) * 4;
    if (i < H) store_norm4(hh, g, i, x[v], inv);
  }
}

__global__ __launch_bounds__(kThreads) void rmsnorm_kernel(const float* __restrict__ r,
                                                           const uint16_t* __restrict__ g,
                                                           uint16_t* __restrict__ h, int H,
                                                           float eps) {
  __shared__ float sh[kThreads / 64];
  const int t = blockIdx.x;
  const float* rr = r + static_cast<int64_t>(t) * H;
  float ss = 0.f;
  for (int i = threadIdx.x * 4; i < H; i += kThreads * 4) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(rr + i);
    ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
  }
  const float inv = rsqrtf(block_sum(ss, sh) / H + eps);
  uint16_t* hh = h + static_cast<int64_t>(t) * H;
  for (int i = threadIdx.x * 4; i < H; i += kThreads * 4)
    store_norm4(hh, g, i, *reinterpret_cast<const f32x4*>(rr + i), inv);
}

}  // namespace

hipError_t launch_embed_rmsnorm(const int32_t* ids, const uint16_t* embed, const uint16_t* gain,
                                float* r, uint16_t* h, int rows, int H, float eps, int vocab,
                                int32_t* err, const RowMap& rm, int d, float theta, float* tab,
                                ClearSpan a, ClearSpan b, const SharedSlots& shared, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int half = d / 2;
  if (half > kThreads) return hipErrorInvalidValue;
  embed_rmsnorm_kernel<<<rows, kThreads, 0, s>>>(ids, embed, gain, r, h, H, eps, vocab, err, rm, half,
                                                 log2(double(theta)) / half, tab, a, b, shared);
  return hipGetLastError();
}

hipError_t launch_rmsnorm(const float* r, const uint16_t* gain, uint16_t* h, int rows, int H,
                          float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (H <= kRegVecs * kThreads * 4)
    rmsnorm_reg_kernel<<<rows, kThreads, 0, s>>>(r, gain, h, H, eps);
  else
    rmsnorm_kernel<<<rows, kThreads, 0, s>>>(r, gain, h, H, eps);
  return hipGetLastError();
}

}  // namespace pallas
