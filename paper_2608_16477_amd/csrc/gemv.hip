// Skinny GEMM for decode (M <= 8 rows): C = X W^T streaming the weights once.
//
// A workgroup of 4 waves owns a tile of TN blocks of 16 weight rows (for the
// gate|up projection half of them gate rows and half the matching up rows)
// and splits K four ways.  Each wave streams its K range in steps of 64: one
// 128-byte line of each weight row and the matching 64 columns of X go
// straight from memory into a private LDS stage with buffer_load ... lds (NS
// stages in flight), each load instruction covering whole lines of 8 rows.
// Inside a stage the 16-byte slots are permuted so the
// v_mfma_f32_16x16x32_bf16 operand reads (16 rows at one k) hit 16 distinct
// bank groups.  The partial tiles of the waves are summed through LDS.
// Launches with too few tiles to fill the chip also split K over workgroups:
// each writes its partial sums with agent-scope stores and counts itself in a
// per-tile counter, and the last to arrive adds the splits in order and
// applies the epilogue (gemv_plan chooses TN and the splits).
//
// More than 8 rows run the GEMM (gemm.hip): X is then a large part of what a
// wave keeps in flight, and the GEMM's tiles share it between waves.  (With two
// blocks of X rows here, decode steps of 9, 12 and 16 rows took 1451, 1521 and
// 1644 us against 1566, 1594 and 1676 through the GEMM at 12 layers of the mid
// model, but 1984, 2133 and 2372 against 1827, 1924 and 2038 at 8 layers of the
// large one; and 9 to 64 rows share the GEMM's K splits, so a row has the same
// bits among any of them.)
//
// Weights are loaded non-temporally: they are read once per step, and the
// stream runs 10% faster that way (M = 1: gate|up of the mid / large model 36
// -> 31.7 / 91 -> 83.2 us, lm_head 202 -> 179 us, 6.9 TB/s).
//
// RMSNorm is folded into the projections on both sides of it.  The residual
// projections (O, down) also write x g (the new residual times the next
// norm's gain, bf16) and the sums of squares of their columns; the projection
// that follows streams x g and scales its rows by (mean(x^2) + eps)^(-1/2).
// bf16 rounding is relative, so x g carries the error of x g / rms, and a
// norm launch of its own (4.6 us, twice per layer) falls away.
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace pallas {

namespace {

constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kRows = kGemvMaxRows;   // rows of X: one block
constexpr int kKStep = 64;        // k per stage: one 128-byte line per row
constexpr int kBlockSlots = 68;   // 8 rows x 8 slots of 16 B, plus 4 slots of padding
constexpr int kAuxAgent = 16;     // buffer cache policy: sc1 (device-coherent)
constexpr int kAuxStream = 2;     // nt
constexpr uint32_t kOob = 0xFFFFFFF0u;

typedef __attribute__((address_space(3))) void lds_void;

// Block slot of (row rr in 0..7, 16-byte chunk c in 0..7).
__device__ __forceinline__ int bslot(int rr, int c) {
  return (rr & 3) + 8 * (rr >> 2) + 4 * (c & 1) + 16 * (c >> 1);
}

struct GemvArgs {
  const uint16_t* X;
  const uint16_t* W;
  void* C;
  int ldx, ldw, ldc, M, N, K;
  int S;          // K splits over workgroups
  float* part;    // partial tiles
  int* ctr;       // [tiles], zero on entry
  GemvNorm nrm;
};

// Sums of squares of X's rows ([part][kRows], four rows per thread): the first
// loads of a thread, started early and not waited for until finish(), then
// (mean(x^2) + eps)^(-1/2) per row.
struct RowScale {
  static constexpr int kQ = kRows / 4;
  static constexpr int U = 4;
  u32x4 x[U];
  __device__ __forceinline__ void load(const GemvNorm& n) {
    const uint32_t bytes = n.ssq_in ? static_cast<uint32_t>(n.parts_in) * (kRows * 4) : 0;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)n.ssq_in, 0, bytes, 0x00020000);
#pragma unroll
    for (int u = 0; u < U; ++u)   // past the end: zeros
      x[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (threadIdx.x + u * kThreads) * 16u, 0, 0));
  }
  // Into row_inv[kRows] through scratch [kWaves][kQ]; every thread calls it.
  // Read row_inv after a barrier.
  __device__ __forceinline__ void finish(const GemvNorm& n, int K, f32x4* scratch, float* row_inv) {
    if (!n.ssq_in) return;
    f32x4 v = {};
#pragma unroll
    for (int u = 0; u < U; ++u) v += __builtin_bit_cast(f32x4, x[u]);
    for (int i = threadIdx.x + U * kThreads; i < n.parts_in * kQ; i += kThreads)
      v += reinterpret_cast<const f32x4*>(n.ssq_in)[i];
#pragma unroll
    for (int o = 32; o >= kQ; o >>= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], o, kWave);
    if ((threadIdx.x & 63) < kQ) scratch[(threadIdx.x >> 6) * kQ + (threadIdx.x & 63)] = v;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (threadIdx.x < kRows) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) s += reinterpret_cast<const float*>(scratch + w * kQ)[threadIdx.x];
      row_inv[threadIdx.x] = rsqrtf(s / K + n.eps);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
};

// NS: stages in flight per wave.
template <int EPI, int TN, int NS>
__global__ __launch_bounds__(kThreads) void gemv_kernel(GemvArgs p) {
  constexpr int kBlocks = 2 * TN + 1;             // load instructions per stage
  constexpr int kStageSlots = kBlocks * kBlockSlots;
  constexpr int HT = TN > 1 ? TN / 2 : 1;         // gate|up: gate blocks of a tile
  constexpr int kRing = kWaves * NS * kStageSlots;
  constexpr int kRed = kWaves * TN * 64;          // partial tiles
  // (one array: see the decode attention kernel's note on LDS waits)
  constexpr int kMain = kRing > kRed ? kRing : kRed;
  __shared__ __attribute__((aligned(16))) u32x4 lds[kMain + (kWaves + 1) * RowScale::kQ + 1];
  f32x4* const scratch = reinterpret_cast<f32x4*>(lds + kMain);
  float* const row_inv = reinterpret_cast<float*>(lds + kMain + kWaves * RowScale::kQ);   // [kRows]
  int* const arrived = reinterpret_cast<int*>(lds + kMain + (kWaves + 1) * RowScale::kQ);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, kg = lane >> 4;
  const int tile = static_cast<int>(blockIdx.x) / p.S, ks = static_cast<int>(blockIdx.x) % p.S;
  const int M = p.M, N = p.N;

  // First weight row of block t, and its first output column.
  auto col0 = [&](int t) { return EPI == kEpiSwiGLU ? (tile * HT + t % HT) * 16 : (tile * TN + t) * 16; };
  auto wrow = [&](int t) { return (EPI == kEpiSwiGLU && t >= HT ? N : 0) + col0(t); };

  // This workgroup's K range [kw0, kw1), then a quarter of it per wave.
  const int kper = ((p.K + p.S * kKStep - 1) / (p.S * kKStep)) * kKStep;
  const int kw0 = ks * kper, kw1 = min(p.K, kw0 + kper);
  const int kslice = ((max(kw1 - kw0, 0) + kWaves * kKStep - 1) / (kWaves * kKStep)) * kKStep;
  const int kb = kw0 + wave * kslice, ke = min(kw1, kb + kslice);
  const int nst = ke > kb ? (ke - kb + kKStep - 1) / kKStep : 0;

  // Load coordinates: a block instruction has lane -> slot lane -> (row rr, chunk c).
  const int b = lane & 15;
  const int rr = (b & 3) | ((b >> 3) << 2);
  const int lc = ((lane >> 4) << 1) | ((b >> 2) & 1);
  const uint32_t woff = static_cast<uint32_t>(rr) * p.ldw * 2u + lc * 16u;
  const uint32_t xoff = static_cast<uint32_t>(rr) * p.ldx * 2u + lc * 16u;
  const __amdgpu_buffer_rsrc_t rx =
      __builtin_amdgcn_make_buffer_rsrc((void*)p.X, 0, static_cast<uint32_t>(M) * p.ldx * 2u, 0x00020000);

  u32x4* const wbase = lds + wave * NS * kStageSlots;
  auto issue = [&](int s) {
    const int k0 = kb + s * kKStep;
    u32x4* st = wbase + (s % NS) * kStageSlots;
    const bool in = k0 + lc * 8 < ke;
    const uint32_t ko = static_cast<uint32_t>(k0) * 2u;
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      // Rows past N: the buffer range ends before them (the count is the
      // same in every lane; kept scalar, so the descriptors are).
      const int valid = __builtin_amdgcn_readfirstlane(max(0, min(16, N - col0(t))));
      const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(p.W + static_cast<int64_t>(valid > 0 ? wrow(t) : 0) * p.ldw), 0,
          static_cast<uint32_t>(valid) * p.ldw * 2u, 0x00020000);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void*)(st + (2 * t + h) * kBlockSlots), 16,
                                                 in ? woff + ko + h * 8u * p.ldw * 2u : kOob, 0, 0, kAuxStream);
    }
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void*)(st + 2 * TN * kBlockSlots), 16, in ? xoff + ko : kOob, 0, 0, 0);
  };

  f32x4 acc[TN];
#pragma unroll
  for (int t = 0; t < TN; ++t) acc[t] = f32x4{0, 0, 0, 0};
  auto compute = [&](int s) {
    const u32x4* st = wbase + (s % NS) * kStageSlots;
#pragma unroll
    for (int q = 0; q < kKStep / 32; ++q) {
      const int sl = bslot(li & 7, 4 * q + kg);
      // (rows 8 to 15 of the operand repeat 0 to 7)
      const bf16x8 a = __builtin_bit_cast(bf16x8, st[2 * TN * kBlockSlots + sl]);
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const bf16x8 w = __builtin_bit_cast(bf16x8, st[(2 * t + (li >> 3)) * kBlockSlots + sl]);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w, acc[t], 0, 0, 0);
      }
    }
  };

  for (int s = 0; s < NS - 1 && s < nst; ++s) issue(s);
  RowScale scale;
  scale.load(p.nrm);
  for (int s = 0; s < nst; ++s) {
    asm volatile("" ::: "memory");
    if (s + NS - 1 < nst) {
      issue(s + NS - 1);
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * kBlocks) : "memory");
    } else if (NS > 2 && nst - 1 - s == 1) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBlocks) : "memory");   // step s + 1 may stay in flight
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    compute(s);
  }
  static_assert(NS == 2 || NS == 3, "the tail leaves at most one step in flight");

  // Epilogue units: block t (gate|up: the pair t, t + HT).  Wave w takes every
  // fourth, from w on.
  constexpr int kT = EPI == kEpiSwiGLU ? HT : TN;     // unit columns per tile
  constexpr int kUnits = (kT + kWaves - 1) / kWaves;  // per wave
  constexpr int kPer = EPI == kEpiSwiGLU ? 2 : 1;     // blocks per unit
  // What the residual epilogue reads, started before the reductions.
  float old[kUnits][4], gain[kUnits];
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    const int t = wave + u * kWaves, col = col0(t) + li;
    gain[u] = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = kg * 4 + r;
      old[u][r] = 0.f;
      if (EPI == kEpiAddF32 && t < kT && col < N && m < M)
        old[u][r] = static_cast<const float*>(p.C)[static_cast<int64_t>(m) * p.ldc + col];
    }
    if (EPI == kEpiAddF32 && p.nrm.gain_out && t < kT && col < N) gain[u] = bf2f(p.nrm.gain_out[col]);
  }
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int t = 0; t < TN; ++t) red[(wave * TN + t) * 64 + lane] = acc[t];
  __syncthreads();
  f32x4 sum[kUnits][kPer];
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    const int t0 = wave + u * kWaves;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int t = t0 + e * HT;
      sum[u][e] = f32x4{};
      if (t0 < kT)
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum[u][e] += red[(w * TN + t) * 64 + lane];
    }
  }
  if (p.S > 1) {
    // Partial tiles in register layout: 16 bytes per lane, whole lines.
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(p.part + static_cast<int64_t>(tile) * p.S * (TN * 256)), 0,
        static_cast<uint32_t>(p.S) * (TN * 1024), 0x00020000);
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int t0 = wave + u * kWaves, t = t0 + e * HT;
        __builtin_amdgcn_raw_buffer_store_b128(
            __builtin_bit_cast(u32x4, sum[u][e]), rp,
            t0 < kT && kg * 4 < M ? static_cast<uint32_t>((ks * TN + t) * 64 + lane) * 16u : kOob,
            0, kAuxAgent);
      }
    // The partials are agent-scope stores, which write through this XCD's L2
    // to the device-coherent level; once every wave's have completed (vmcnt
    // 0, barrier), the count goes up.  The reader's agent-scope loads miss
    // its own L2, and are issued only after the count they branch on has
    // returned.  That is the agent-scope release/acquire sequence of the
    // gfx950 memory model for data accessed only at agent scope: its L2
    // write-back and invalidate act on other data only, and as fences
    // (__ATOMIC_RELEASE / __ATOMIC_ACQUIRE at agent scope) they cost a whole
    // L2 per workgroup: measured, a decode step of the large model took 21.6
    // ms with them against 14.9 ms.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (threadIdx.x == 0)
      *arrived = __hip_atomic_fetch_add(p.ctr + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (*arrived != p.S - 1) return;
    if (threadIdx.x == 0) __hip_atomic_store(p.ctr + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Last of the tile: every split's partials at once, added in order.
#pragma unroll
    for (int u = 0; u < kUnits; ++u)
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int t0 = wave + u * kWaves, t = t0 + e * HT;
        f32x4 v[kGemvMaxSplit];
#pragma unroll
        for (int j = 0; j < kGemvMaxSplit; ++j)     // past S: reads zeros
          v[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
              rp, j < p.S && t0 < kT ? static_cast<uint32_t>((j * TN + t) * 64 + lane) * 16u : kOob, 0,
              kAuxAgent));
        sum[u][e] = v[0];
#pragma unroll
        for (int j = 1; j < kGemvMaxSplit; ++j)
          if (j < p.S) sum[u][e] += v[j];
      }
  }
  float inv[4] = {1.f, 1.f, 1.f, 1.f};
  if (p.nrm.ssq_in) {
    scale.finish(p.nrm, p.K, scratch, row_inv);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int r = 0; r < 4; ++r) inv[r] = row_inv[min(kg * 4 + r, kRows - 1)];
  }
  // lane holds column li and rows 4 kg + r
  float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < kUnits; ++u) {
    const int t = wave + u * kWaves;
    const int col = col0(t) + li;
    if (t >= kT || col >= N) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = kg * 4 + r;
      if (m >= M) continue;
      const int64_t at = static_cast<int64_t>(m) * p.ldc + col;
      const float v = sum[u][0][r] * inv[r];
      if (EPI == kEpiSwiGLU) {
        static_cast<uint16_t*>(p.C)[at] = f2bf(swiglu(v, sum[u][kPer - 1][r] * inv[r]));
      } else if (EPI == kEpiBf16) {
        static_cast<uint16_t*>(p.C)[at] = f2bf(v);
      } else if (EPI == kEpiAddF32) {
        const float x = old[u][r] + v;
        static_cast<float*>(p.C)[at] = x;
        if (p.nrm.gain_out) {
          p.nrm.h_out[at] = f2bf(x * gain[u]);
          ss[r] += x * x;
        }
      } else {
        static_cast<float*>(p.C)[at] = v;
      }
    }
  }
  if (EPI == kEpiAddF32 && p.nrm.gain_out && wave < kT) {
    // One partial per row and wave of the tile that covers it.
    f32x4 sq;
#pragma unroll
    for (int r = 0; r < 4; ++r) sq[r] = row16_sum(ss[r]);
    if (li == 0 && kg * 4 < kRows)
      *reinterpret_cast<f32x4*>(p.nrm.ssq_out +
                                (static_cast<int64_t>(tile) * kT + wave) * kRows + kg * 4) = sq;
  }
}

template <int EPI>
hipError_t launch_epi(const GemvArgs& a, const GemvPlan& pl, int grid, hipStream_t s) {
  if (pl.tn == 2) gemv_kernel<EPI, 2, 2><<<grid, kThreads, 0, s>>>(a);
  else if (pl.tn == 4) gemv_kernel<EPI, 4, 2><<<grid, kThreads, 0, s>>>(a);
  else if constexpr (EPI != kEpiSwiGLU) gemv_kernel<EPI, 1, 3><<<grid, kThreads, 0, s>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemv(int epi, const uint16_t* A, int lda, const uint16_t* B, int ldb, void* C, int ldc, int M, int N,
                       int K, const GemvScratch& sc, const GemvNorm& nrm, hipStream_t s) {
  if (M <= 0 || M > kGemvMaxRows || N <= 0 || K <= 0 || (K & 7) || (lda & 7) || (ldb & 7)) return hipErrorInvalidValue;
  // 32-bit buffer offsets: 16 weight rows and the X rows
  if (static_cast<int64_t>(16) * ldb * 2 >= (int64_t(1) << 32) || static_cast<int64_t>(kGemvMaxRows) * lda * 2 >= (int64_t(1) << 32))
    return hipErrorInvalidValue;
  const GemvPlan pl = gemv_plan(epi, N, K);
  if (pl.counters() > sc.ctr_count || pl.part_bytes() > sc.part_bytes) return hipErrorInvalidValue;
  GemvArgs a;
  a.X = A;
  a.W = B;
  a.C = C;
  a.ldx = lda;
  a.ldw = ldb;
  a.ldc = ldc;
  a.M = M;
  a.N = N;
  a.K = K;
  a.S = pl.S;
  a.part = sc.part;
  a.ctr = sc.ctr;
  a.nrm = nrm;
  const int grid = pl.tiles * pl.S;
  switch (epi) {
    case kEpiBf16: return launch_epi<kEpiBf16>(a, pl, grid, s);
    case kEpiAddF32: return launch_epi<kEpiAddF32>(a, pl, grid, s);
    case kEpiF32: return launch_epi<kEpiF32>(a, pl, grid, s);
    case kEpiSwiGLU: return launch_epi<kEpiSwiGLU>(a, pl, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pallas
