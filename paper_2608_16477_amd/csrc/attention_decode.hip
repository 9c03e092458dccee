// Decode attention over the paged KV cache, one query row per sequence:
// QK-norm and rotary of the row's Q and K, the paged store of its K and V,
// grouped-query attention over positions [0, n], in one kernel.
//
// A sequence's keys are cut into splits of a length that its own position
// gives (decode_split_keys), and each split into four leaves.  A leaf is one
// online softmax over its 32-key blocks in order; leaves are merged as a
// binary tree.  A workgroup of two or four waves owns a run of splits of one
// (sequence, KV head) and all G query heads that share it, and its waves equal
// shares of the run's leaves.  Runs are aligned parts of the tree, so how many
// splits a run has, and how many waves, changes no bit: a sequence's result
// does not depend on the others in the call, though the division of the work
// does (plan_decode_runs).
//
// Each wave walks its blocks on its own: K and V rows go from memory straight
// into a private two-stage LDS ring (buffer_load ... lds, whole 256-byte head
// rows), so up to 32 KiB per wave and 128 KiB per CU are in flight and the
// waves meet no barrier until the end.
//
// Scores are S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (the G heads are the
// columns, repeated up to 16): lane l holds keys 4 (l / 16) + r of head l mod 16.
// O^T = V^T P^T takes those registers as its B operand as they are, with V
// read transposed from LDS (ds_read_b64_tr_b16).  P stays 32-bit: it is
// split into three bf16 parts whose sum is P exactly, one MFMA each; the
// matrix cores are idle here, and the kernel is bound by the K/V stream.
//
// A row may attend to slots that other rows of the call write (several tokens
// of one sequence, a table that another row's reaches).  Those rows' stores
// come from other workgroups of this launch, in no order, so such keys are
// taken from the rows' projections instead: the result is that of storing
// every row's K and V before any attention.  The call's start launch flags the
// rows that do.
//
// Runs are merged by the last workgroup of a (sequence, KV head) to
// arrive: partial records and an arrival count through agent-scope accesses,
// as the skinny projections do.
//
// Per layer against the three kernels this replaces (norm / rotary / store,
// 64-key splits on the vector units, merge): 32 sequences of 136,000 keys in
// all, 8 KV heads of 128 (558 MB): 213 -> 109 us (5.1 TB/s; bound by the K/V
// stream); 8 sequences, 32,000 keys: 69 -> 32 us; one sequence of 4000 keys,
// 64 query heads: 27 -> 12 us (bound by the chain of launch, table, stream,
// record store, count and merge).  Runs of equal length over all sequences,
// whose merges depend on the batch, take 106, 31.7 and 12.1 us; 16 and 64
// sequences of 500 to 8000 keys, 64 query heads, 29.2 against 31.8 and 136
// against 145 us.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace pallas {

namespace {

constexpr int kPage = 16;        // tokens per cache page (the only page size the library accepts)
// The declared bound is above the launched 128 or 256: it limits a wave to 256
// registers, and the compiler then keeps the accumulators in vector registers
// (with 512 it moves them to accumulation registers and back in every block).
constexpr int kBoundThreads = 512;
constexpr int kBlk = 32;         // keys per block: two pages
constexpr int kStages = 2;       // blocks in flight per wave
constexpr int kAuxAgent = 16;    // buffer cache policy: sc1 (device-coherent)
constexpr int kAuxStream = 2;    // nt: K and V are read once per step

typedef __attribute__((address_space(3))) void lds_void;

// LDS rows are whole head rows of CH 16-byte chunks; chunk c of row r sits in
// slot c ^ swz(r).  K: the 16 rows an MFMA operand read covers at one chunk
// land on 16 distinct 4-bank groups.  V: the 8 keys x 2 chunks that half of a
// transposed read covers do.
template <int CH>
__device__ __forceinline__ int swz_k(int row) { return CH == 16 ? row & 15 : (row >> 1) & 7; }
template <int CH>
__device__ __forceinline__ int swz_v(int row) { return CH == 16 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); }

// Four output tiles of the PV operand from a V block at LDS byte address
// `vb`: keys 4 q4 .. + 3 of its first page (at the tile's address, vb XOR 32
// per tile) and of its second (`kSecond` bytes further).  In each 16-lane
// group, ds_read_b64_tr_b16 hands lane i element i % 4 of the 64-bit words
// read by lanes i / 4, i / 4 + 4, i / 4 + 8 and i / 4 + 12: four consecutive
// keys of one dimension.  Reads and their wait are one statement: before the
// builtin form of this read the compiler waits for every load in flight into
// LDS, which would empty the ring at each block.
template <int kSecond>
__device__ __forceinline__ void read_pv4(uint32_t vb, int dt0, u32x4* a) {
  const uint32_t x0 = vb ^ ((dt0 + 0) * 32u), x1 = vb ^ ((dt0 + 1) * 32u);
  const uint32_t x2 = vb ^ ((dt0 + 2) * 32u), x3 = vb ^ ((dt0 + 3) * 32u);
  u32x2 l0, l1, l2, l3, h0, h1, h2, h3;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %9\n\t"
      "ds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\t"
      "ds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
      "ds_read_b64_tr_b16 %6, %11\n\t"
      "ds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(l0), "=&v"(h0), "=&v"(l1), "=&v"(h1), "=&v"(l2), "=&v"(h2), "=&v"(l3), "=&v"(h3)
      : "v"(x0), "v"(x1), "v"(x2), "v"(x3), "n"(kSecond)
      : "memory");
  a[0] = u32x4{l0.x, l0.y, h0.x, h0.y};
  a[1] = u32x4{l1.x, l1.y, h1.x, h1.y};
  a[2] = u32x4{l2.x, l2.y, h2.x, h2.y};
  a[3] = u32x4{l3.x, l3.y, h3.x, h3.y};
}

// Max / sum over the four 16-lane rows of a wave (lanes l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float rows_max(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float rows_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// (a, b) as packed bf16, and what is left of them.
__device__ __forceinline__ uint32_t take_bf2(float& a, float& b) {
  const uint32_t w = pack_bf2(a, b);
  a -= bflo(w);
  b -= bfhi(w);
  return w;
}

// A partial softmax: exponentials relative to the maximum m that sum to l, and
// (beside it) a weighted sum of V.  Merging with an empty one (m -inf, zeros)
// changes no bit, and the fused multiply-adds are written out, so every caller
// rounds alike.
struct Partial {
  float m, l;
};
struct Weights {
  float a, b;
};
__device__ __forceinline__ Partial merge(Partial a, Partial b, Weights& w) {
  const float m = fmaxf(a.m, b.m);
  w.a = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(a.m - m);
  w.b = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(b.m - m);
  return {m, __builtin_fmaf(w.b, b.l, w.a * a.l)};
}
__device__ __forceinline__ f32x4 merge(f32x4 a, f32x4 b, Weights w) {
  f32x4 v;
#pragma unroll
  for (int x = 0; x < 4; ++x) v[x] = __builtin_fmaf(w.b, b[x], w.a * a[x]);
  return v;
}

// The N (a power of two) partials as a binary tree, into the first.
template <int N>
__device__ __forceinline__ void merge_tree(Partial* ml, f32x4* v) {
#pragma unroll
  for (int d = 1; d < N; d *= 2)
#pragma unroll
    for (int k = 0; k < N; k += 2 * d) {
      Weights w;
      ml[k] = merge(ml[k], ml[k + d], w);
      v[k] = merge(v[k], v[k + d], w);
    }
}

// Loads of the run's 32-key block `blk` (below nblk) into a stage: cached
// rows only (positions below n, `cached` of them from the run's start); the
// others, and rows on a page outside the pool, read zeros, as do blocks from
// nblk on.  Every wave issues the loads of every step, so the compiler
// can count the loads in flight.  koff / voff: byte offset
// in a page of what this lane loads in instruction v of it.
template <int D>
__device__ __forceinline__ void issue_block(const DecodeAttnParams& p, int kh, int entry, int cached, int blk, int nblk,
                                            uint32_t rs, const uint32_t* koff, const uint32_t* voff, u32x4* st) {
  constexpr int CH = D / 8, IPP = kPage / (64 / CH);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int pg = blk < nblk ? __builtin_amdgcn_readlane(entry, blk * 2 + h) : -1;
    const int nv = min(kPage, cached - (blk * kBlk + h * kPage));
    const uint32_t range = pg >= 0 && nv > 0 ? static_cast<uint32_t>(nv - 1) * rs + D * 2 : 0;
    const int64_t base = (static_cast<int64_t>(max(pg, 0)) * kPage * p.Hkv + kh) * D;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(p.k_plane + base), 0, range, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(p.v_plane + base), 0, range, 0x00020000);
#pragma unroll
    for (int v = 0; v < IPP; ++v)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void*)(st + (h * IPP + v) * 64), 16, koff[v], 0, 0, kAuxStream);
#pragma unroll
    for (int v = 0; v < IPP; ++v)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(st + kBlk * CH + (h * IPP + v) * 64), 16, voff[v], 0, 0, kAuxStream);
  }
}

// K (normalised and rotated) and V of row `row` of the call, as key `r` of the
// 32-key block in stage Kst, Vst.  Rare: kept out of the stream's registers.
template <int D>
__device__ __forceinline__ void put_row(const DecodeAttnParams& p, int kh, int row, int r, u32x4* Kst, u32x4* Vst) {
  constexpr int CH = D / 8, LPH = D / 8, HALF = D / 2;
  const int lane = threadIdx.x & 63, j = lane % LPH;
  if (lane >= 2 * LPH) return;                  // lanes [0, LPH): K, [LPH, 2 LPH): V
  const bool isk = lane < LPH;
  const uint16_t* src = p.qkv + static_cast<int64_t>(row) * p.qkv_ld +
                        static_cast<int64_t>(p.Hq + (isk ? 0 : p.Hkv) + kh) * D;
  u32x2 lo = *reinterpret_cast<const u32x2*>(src + 4 * j), hi = *reinterpret_cast<const u32x2*>(src + HALF + 4 * j);
  if (isk) {
    u32x2 g0{}, g1{};
    if (p.qk_norm) {
      g0 = *reinterpret_cast<const u32x2*>(p.k_gain + 4 * j);
      g1 = *reinterpret_cast<const u32x2*>(p.k_gain + HALF + 4 * j);
    }
    const f32x4* rope = reinterpret_cast<const f32x4*>(p.rope + (static_cast<int64_t>(row) * HALF + 4 * j) * 2);
    norm_rope4<D>(lo, hi, p.qk_norm, g0, g1, p.eps, rope[0], rope[1]);
  }
  u32x4* st = isk ? Kst : Vst;
  const int swz = isk ? swz_k<CH>(r) : swz_v<CH>(r), c = j / 2;
  reinterpret_cast<u32x2*>(st + r * CH + (c ^ swz))[j % 2] = lo;
  reinterpret_cast<u32x2*>(st + r * CH + ((c + CH / 2) ^ swz))[j % 2] = hi;
}

template <int D, int kWaves>
__global__ __launch_bounds__(kBoundThreads) void attn_decode_kernel(DecodeAttnParams p, RowMap rm, DecodeRuns runs,
                                                               float* __restrict__ part_o,
                                                               float* __restrict__ part_ml, int* __restrict__ ctr) {
  constexpr int kThreads = kWaves * 64;
  constexpr int kLevels = kWaves == 2 ? 3 : 2;  // a wave merges up to 2^kLevels leaves
  constexpr int CH = D / 8;                     // 16-byte chunks per row
  constexpr int RPI = 64 / CH;                  // rows per load instruction
  constexpr int IPP = kPage / RPI;              // load instructions per page
  constexpr int kStageSlots = kBlk * CH;        // 16-byte slots of a K or V block
  constexpr int LPH = D / 8;                    // lanes per head in the norm / rotary pass
  constexpr int HALF = D / 2;
  constexpr int HPP = kThreads / LPH;           // heads per pass
  constexpr int kHeadsMax = 10;                 // G <= 8 query heads, K, V
  constexpr int NPASS = (kHeadsMax + HPP - 1) / HPP;
  constexpr int DT = D / 16;                    // output tiles
  // One array: with several, the compiler's alias scopes make LDS reads of a
  // stage wait for the loads in flight into the other.
  constexpr int kRingSlots = kWaves * kStages * 2 * kStageSlots;
  __shared__ __attribute__((aligned(256))) u32x4 lds[kRingSlots + kHeadsMax * CH + kWaves * 4 + 1];
  uint16_t(*heads)[D] = reinterpret_cast<uint16_t(*)[D]>(lds + kRingSlots);   // Q heads, then K and V of this row
  Partial(*wave_ml)[8] = reinterpret_cast<Partial(*)[8]>(lds + kRingSlots + kHeadsMax * CH);   // [wave][head]
  int* arrived = reinterpret_cast<int*>(lds + kRingSlots + kHeadsMax * CH + kWaves * 4);

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int q4 = lane >> 4, l16 = lane & 15;
  const int G = p.Hq / p.Hkv;
  const int kh = static_cast<int>(blockIdx.x) % p.Hkv, u = static_cast<int>(blockIdx.x) / p.Hkv;
  int s = 0, hi = rm.n_seqs - 1;                // largest s with first[s] <= u
  while (s < hi) {
    const int mid = (s + hi + 1) >> 1;
    if (runs.first[mid] <= u) s = mid; else hi = mid - 1;
  }
  const int run = u - runs.first[s], nrun = runs.first[s + 1] - runs.first[s];
  const int n = rm.base_pos[s], row = rm.cu[s];
  const int split_keys = decode_split_keys(n), run_keys = runs.per_run[s] * split_keys;
  const int j0 = run * run_keys;
  const int j1 = min(j0 + run_keys, n + 1);
  const bool last = run == nrun - 1;            // holds position n
  const int32_t* bt = p.bt + static_cast<int64_t>(s) * p.max_pages;
  int shared = rm.n_seqs > 1 ? p.shared[s] : 0;

  // This run's table entries, one per lane (a run is at most 64 pages).
  int entry = -1;
  {
    const int pi = j0 / kPage + lane;
    if (pi * kPage < j1) entry = bt[pi];
    if (entry < 0 || entry >= p.num_pages) entry = -1;
  }
  // The row's Q heads (and K and V heads): a lane owns rotary pairs 4 j .. 4 j + 3.
  const int j = t % LPH, hsub = t / LPH;
  u32x2 lov[NPASS], hiv[NPASS];
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) {
    const int hs = ps * HPP + hsub;
    lov[ps] = hiv[ps] = u32x2{0, 0};
    if (hs < G + (last ? 2 : 0)) {
      const int hh = hs < G ? kh * G + hs : p.Hq + (hs - G) * p.Hkv + kh;
      const uint16_t* src = p.qkv + static_cast<int64_t>(row) * p.qkv_ld + static_cast<int64_t>(hh) * D;
      lov[ps] = *reinterpret_cast<const u32x2*>(src + 4 * j);
      hiv[ps] = *reinterpret_cast<const u32x2*>(src + HALF + 4 * j);
    }
  }
  // Gains of Q and K and the rotary factors: loaded, and waited for with the
  // table entries, before the K/V stream (loads return in order).
  u32x2 gq[2] = {}, gk[2] = {};
  if (p.qk_norm) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      gq[e] = *reinterpret_cast<const u32x2*>(p.q_gain + e * HALF + 4 * j);
      gk[e] = *reinterpret_cast<const u32x2*>(p.k_gain + e * HALF + 4 * j);
    }
  }
  const f32x4* rope = reinterpret_cast<const f32x4*>(p.rope + (static_cast<int64_t>(row) * HALF + 4 * j) * 2);
  f32x4 cs01 = rope[0], cs23 = rope[1];         // (cos, sin) of pairs 4j .. 4j+3
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) asm volatile("" : "+v"(lov[ps]), "+v"(hiv[ps]));
  asm volatile("" : "+v"(cs01), "+v"(cs23), "+v"(gq[0]), "+v"(gq[1]), "+v"(gk[0]), "+v"(gk[1]), "+v"(entry));

  // The run's leaves (a quarter of a split each) in order, as many per wave.
  const int leaf_blocks = split_keys / (4 * kBlk), leaves = runs.per_run[s] * (4 / kWaves);
  const int blk0 = wave * leaves * leaf_blocks;  // this wave's blocks: [blk0, blk1)
  const int blk1 = min(blk0 + leaves * leaf_blocks, (j1 - j0 + kBlk - 1) / kBlk);
  u32x4* const myring = lds + wave * kStages * 2 * kStageSlots;   // [stage][K, V]
  const uint32_t rs = static_cast<uint32_t>(p.Hkv) * D * 2;   // bytes between tokens of a page
  // Byte offset in a page of what this lane loads in instruction v of it.
  uint32_t koff[IPP], voff[IPP];
#pragma unroll
  for (int v = 0; v < IPP; ++v) {
    const int r = v * RPI + lane / CH;
    koff[v] = r * rs + static_cast<uint32_t>(((lane % CH) ^ swz_k<CH>(r)) * 16);
    voff[v] = r * rs + static_cast<uint32_t>(((lane % CH) ^ swz_v<CH>(r)) * 16);
  }
  constexpr int kLoads = 4 * IPP;               // load instructions per block
  issue_block<D>(p, kh, entry, n - j0, blk0, blk1, rs, koff, voff, myring);
  issue_block<D>(p, kh, entry, n - j0, blk0 + 1, blk1, rs, koff, voff, myring + 2 * kStageSlots);

  // QK-norm and rotary of Q (and, in the last run, of K).
#pragma unroll
  for (int ps = 0; ps < NPASS; ++ps) {
    const int hs = ps * HPP + hsub;
    if (hs >= G + (last ? 2 : 0)) continue;
    u32x2 olo = lov[ps], ohi = hiv[ps];
    if (hs <= G) norm_rope4<D>(olo, ohi, p.qk_norm, hs < G ? gq[0] : gk[0], hs < G ? gq[1] : gk[1], p.eps, cs01, cs23);
    *reinterpret_cast<u32x2*>(&heads[hs][4 * j]) = olo;
    *reinterpret_cast<u32x2*>(&heads[hs][HALF + 4 * j]) = ohi;
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

  bf16x8 qf[D / 32];
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk)
    qf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(&heads[l16 % G][kk * 32 + q4 * 8]));

  // Slot in a K block (row l16, chunk q4) and byte offset in a V block (key
  // 4 q4 + l16 / 4, dimensions 4 (l16 % 4) ..): substep kk is XOR 4 kk,
  // output tile dt XOR 32 dt, the block's second page + 16 rows.
  const uint32_t kb0 = static_cast<uint32_t>(l16 * CH + (q4 ^ swz_k<CH>(l16)));
  const int vkey = 4 * q4 + (l16 >> 2);
  const uint32_t vb0 = static_cast<uint32_t>(vkey * D * 2 + ((swz_v<CH>(vkey) | ((l16 & 3) >> 1)) * 16) + (l16 & 1) * 8);

  // Rare: cached slots of this run that a row of this call writes (bit r of lane
  // l: slot r of the run's page l).  Their K/V may not be in the pool yet: they
  // are taken from that row, as if every row had stored its own first.  (Lane
  // i: the position that row i writes, and its page.)
  uint32_t fresh = 0;
  int wpos = 0, wpage = -1;
  if (shared) {
    if (lane < rm.n_seqs) {
      wpos = rm.base_pos[lane];
      wpage = p.bt[static_cast<int64_t>(lane) * p.max_pages + wpos / kPage];
    }
    for (int i = 0; i < rm.n_seqs; ++i) {
      const int pg = __builtin_amdgcn_readlane(wpage, i), r = __builtin_amdgcn_readlane(wpos, i) % kPage;
      if (entry == pg) fresh |= 1u << r;
    }
    const int cached = max(0, min(kPage, n - j0 - lane * kPage));
    fresh = entry < 0 ? 0 : fresh & ((1u << cached) - 1);
  }
  const bool any_fresh = __builtin_amdgcn_ballot_w64(fresh != 0) != 0;

  // Leaves are merged as a binary counter counts: held[v] is the merge of 2^v
  // leaves that waits for the next 2^v.  (Set before they are read.)
  f32x4 acc[DT], held[kLevels][DT];
  Partial ml, held_ml[kLevels];
  int blk = blk0;
#pragma unroll 1
  for (int leaf = 0; leaf < leaves; ++leaf) {
  const int end = min(blk0 + (leaf + 1) * leaf_blocks, blk1);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = f32x4{};
  float m = -INFINITY, lsum = 0.f;
  for (; blk < end; ++blk) {
    u32x4* const Kst = myring + (static_cast<unsigned>(blk - blk0) % kStages) * 2 * kStageSlots;
    u32x4* const Vst = Kst + kStageSlots;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");   // this block is here, the next may not be
    const int jb = j0 + blk * kBlk;
    const int pg0 = __builtin_amdgcn_readlane(entry, blk * 2), pg1 = __builtin_amdgcn_readlane(entry, blk * 2 + 1);
    if (any_fresh) {
      for (int h = 0; h < 2; ++h) {
        const int pg = h ? pg1 : pg0;
        for (uint32_t bits = __builtin_amdgcn_readlane(fresh, blk * 2 + h); bits; bits &= bits - 1) {
          const int r = __builtin_ctz(bits);
          const int from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(wpage == pg && wpos % kPage == r));
          put_row<D>(p, kh, rm.cu[from], h * kPage + r, Kst, Vst);
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    if (n - jb < kBlk) {
      // Position n is in this block: its K and V come from this row.
      const int r = n - jb;
      if (lane < 2 * CH) {
        const int c = lane % CH;
        const bool isk = lane < CH;
        const u32x4 x = *reinterpret_cast<const u32x4*>(&heads[isk ? G : G + 1][c * 8]);
        if (isk) Kst[r * CH + (c ^ swz_k<CH>(r))] = x;
        else Vst[r * CH + (c ^ swz_v<CH>(r))] = x;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    f32x4 sc[2] = {f32x4{}, f32x4{}};
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bf16x8 a = __builtin_bit_cast(
            bf16x8, Kst[(kb0 ^ (kk * 4u)) + h * (kPage * CH)]);
        sc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[kk], sc[h], 0, 0, 0);
      }
    u32x4 va[DT];
    const uint32_t vst = vb0 + static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void*)Vst));
#pragma unroll
    for (int dt = 0; dt < DT; dt += 4) read_pv4<kPage * D * 2>(vst, dt, va + dt);
    float pr[8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) pr[h * 4 + r] = sc[h][r] * p.scale_log2;
    if (n - jb < kBlk - 1 || pg0 < 0 || pg1 < 0) {
      // Keys past n, and keys on a page outside the pool.
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (jb + h * kPage + 4 * q4 + r > n || (h ? pg1 : pg0) < 0) pr[h * 4 + r] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(fmaxf(pr[0], pr[1]), fmaxf(pr[2], pr[3])), fmaxf(fmaxf(pr[4], pr[5]), fmaxf(pr[6], pr[7])));
    mx = rows_max(mx);
    if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
      const float m_new = fmaxf(m, mx);
      const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] *= alpha;
    }
    const float mc = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pr[e] = __builtin_amdgcn_exp2f(pr[e] - mc);
      lsum += pr[e];
    }
    bf16x8 pb[3];
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = take_bf2(pr[2 * e], pr[2 * e + 1]);
      pb[part] = __builtin_bit_cast(bf16x8, w);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int part = 2; part >= 0; --part)
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, va[dt]), pb[part], acc[dt], 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this block's LDS reads are done
    issue_block<D>(p, kh, entry, n - j0, blk + kStages, blk1, rs, koff, voff, Kst);
  }
  ml = {m, rows_sum(lsum)};
  bool carry = true;
#pragma unroll
  for (int v = 0; v < kLevels; ++v) {
    carry = carry && (2 << v) <= leaves;
    if (carry && (leaf >> v & 1)) {
      Weights w;
      ml = merge(held_ml[v], ml, w);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[dt] = merge(held[v][dt], acc[dt], w);
    } else if (carry) {
      held_ml[v] = ml;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) held[v][dt] = acc[dt];
      carry = false;
    }
  }
  }

  if (last && t < 2 * CH) {
    // K and V of position n (stored here: a store pending in the loop would
    // make its waits drain every load).
    const int pg = __builtin_amdgcn_readlane(entry, (n - j0) / kPage);
    if (pg >= 0) {
      uint16_t* dst = (t < CH ? p.k_plane : p.v_plane) +
                      ((static_cast<int64_t>(pg) * kPage + n % kPage) * p.Hkv + kh) * D + (t % CH) * 8;
      *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(&heads[t < CH ? G : G + 1][(t % CH) * 8]);
    } else if (t % CH == 0 && p.err) {
      atomicOr(p.err, static_cast<int32_t>(PALLAS_DEVERR_PAGE));
    }
  }

  // Merge the waves through LDS (the ring is free once all are here and
  // nothing is in flight): om[wave][head][dim].
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  float* om = reinterpret_cast<float*>(lds);
  if (l16 < G) {
    float* dst = om + (wave * 8 + l16) * D + 4 * q4;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<f32x4*>(dst + dt * 16) = acc[dt];
    if (q4 == 0) wave_ml[wave][l16] = ml;
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  const int quads = G * D / 4;                  // 4-wide output groups of this KV head
  uint16_t* orow = p.o + (static_cast<int64_t>(row) * p.Hq + kh * G) * D;
  auto store_out = [&](int e, f32x4 v, float l) {
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] = l > 0.f ? v[x] / l : 0.f;
    u32x2 w;
    w.x = pack_bf2(v[0], v[1]);
    w.y = pack_bf2(v[2], v[3]);
    *reinterpret_cast<u32x2*>(orow + e * 4) = w;
  };
  const int64_t rec0 = (static_cast<int64_t>(s) * p.Hkv + kh) * runs.most;   // this (sequence, KV head)'s records
  const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(part_o + rec0 * G * D), 0, static_cast<uint32_t>(runs.most * G * D * 4), 0x00020000);
  Partial* rec_ml = reinterpret_cast<Partial*>(part_ml) + rec0 * G;   // [run][head]
  for (int e = t; e < quads; e += kThreads) {
    const int g = e / (D / 4), dv = (e % (D / 4)) * 4;
    Partial pm[kWaves];
    f32x4 pv[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      pm[w] = wave_ml[w][g];
      pv[w] = *reinterpret_cast<const f32x4*>(om + (w * 8 + g) * D + dv);
    }
    merge_tree<kWaves>(pm, pv);
    if (nrun == 1) {
      store_out(e, pv[0], pm[0].l);
    } else {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, pv[0]), ro, (run * G * D + e * 4) * 4, 0, kAuxAgent);
      if (dv == 0) {
        __hip_atomic_store(&rec_ml[run * G + g].m, pm[0].m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&rec_ml[run * G + g].l, pm[0].l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (nrun == 1) return;
  // Every wave's records have reached the device-coherent level (agent-scope
  // stores write through; vmcnt 0), then the count goes up; the last of the
  // (sequence, KV head) reads the others' past its own L2.
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  int* cnt = ctr + s * p.Hkv + kh;
  if (t == 0) *arrived = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (*arrived != nrun - 1) return;
  if (t == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // All records of a batch of runs are in flight at once, for each of this
  // thread's E output groups.  A batch is an aligned part of the tree.
  constexpr int E = (8 * D / 4 + kThreads - 1) / kThreads, U = E == 1 ? kDecodeSplitsPerSeq : kDecodeSplitsPerSeq / 2;
  const __amdgpu_buffer_rsrc_t rml = __builtin_amdgcn_make_buffer_rsrc(
      (void*)rec_ml, 0, static_cast<uint32_t>(nrun * G * 8), 0x00020000);
  Partial total[E];
  f32x4 v[E];
#pragma unroll
  for (int x = 0; x < E; ++x) {
    total[x] = {-INFINITY, 0.f};
    v[x] = f32x4{};
  }
  for (int k0 = 0; k0 < nrun; k0 += U) {
    f32x4 o[E][U];
    Partial a[E][U];
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
      for (int x = 0; x < E; ++x) {
        const int e = x * kThreads + t, g = e / (D / 4);
        const bool in = k0 + k < nrun && e < quads;        // else: reads zeros
        const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
            rml, in ? ((k0 + k) * G + g) * 8 : 0xFFFFFFF0u, 0, kAuxAgent));
        a[x][k] = {__uint_as_float(r.x), __uint_as_float(r.y)};
        o[x][k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
            ro, in ? ((k0 + k) * G * D + e * 4) * 4 : 0xFFFFFFF0u, 0, kAuxAgent));
      }
#pragma unroll
    for (int x = 0; x < E; ++x) {
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (k0 + k >= nrun) a[x][k].m = -INFINITY;
      merge_tree<U>(a[x], o[x]);
      Weights w;
      total[x] = merge(total[x], a[x][0], w);   // (the first batch: with an empty one)
      v[x] = merge(v[x], o[x][0], w);
    }
  }
#pragma unroll
  for (int x = 0; x < E; ++x)
    if (x * kThreads + t < quads) store_out(x * kThreads + t, v[x], total[x].l);
}

}  // namespace

// How the work is divided (us per layer; 8 KV heads of 128, 4 or 8 query heads
// per KV head).
//   Up to one workgroup per CU, in runs of at most 512 keys: four waves in each
// (one sequence of 2048 keys 10.9 against 12.4 with two; 4 sequences, 13,900
// keys, 18.0 in 224 workgroups, 25 in the 376 that one split each would make).
//   Else two waves, two workgroups to a CU (their starts and merges overlap the
// other's stream), and the fewest whole rounds of them that runs of up to 1024
// keys and four splits allow, filled by doubling the shortest runs only as
// often as needed: 8 sequences 31.9 in 512 workgroups, 35.4 in 800, 39.6 in
// 376; 16 sequences 31.4 in 504, 35 in 416 and in 976.
constexpr int kCus = 256;

bool plan_decode_runs(const RowMap& rm, int Hkv, DecodeRuns& runs) {
  if (rm.n_seqs < 1 || rm.n_seqs > kMaxSeqs) return false;
  for (int i = 0; i < rm.n_seqs; ++i)
    if (rm.base_pos[i] < 0 || decode_split_keys(rm.base_pos[i]) > kDecodeMaxRun) return false;
  int split_keys[kMaxSeqs], splits[kMaxSeqs];
  for (int i = 0; i < rm.n_seqs; ++i) {
    split_keys[i] = decode_split_keys(rm.base_pos[i]);
    splits[i] = rm.base_pos[i] / split_keys[i] + 1;
  }
  auto count = [&](int i) { return (splits[i] + runs.per_run[i] - 1) / runs.per_run[i]; };
  int64_t wgs;
  auto start = [&] {
    wgs = 0;
    for (int i = 0; i < rm.n_seqs; ++i) {
      runs.per_run[i] = 1;
      wgs += int64_t(splits[i]) * Hkv;
    }
  };
  // Doubles the shortest runs that may have up to `keys` keys until at most
  // `most` workgroups are left (the shortest first: a doubled run's turn comes
  // at its new length).
  auto grow = [&](int64_t most, int keys) {
    for (int r = kDecodeMinSplit; 2 * r <= keys; r += kDecodeMinSplit)
      for (int i = 0; i < rm.n_seqs && wgs > most; ++i) {
        const int c = count(i);
        if (split_keys[i] * runs.per_run[i] != r || 2 * runs.per_run[i] > kDecodeMaxRunSplits || c == 1) continue;
        runs.per_run[i] *= 2;
        wgs -= int64_t(c - count(i)) * Hkv;
      }
  };
  start();
  grow(kCus, kDecodeMaxRun / 2);
  runs.wide = wgs <= kCus;
  if (!runs.wide) {
    start();
    grow(0, kDecodeMaxRun);
    const int64_t full = (wgs + 2 * kCus - 1) / (2 * kCus) * (2 * kCus);
    start();
    grow(full, kDecodeMaxRun);
  }
  runs.first[0] = 0;
  runs.most = 1;
  for (int i = 0; i < rm.n_seqs; ++i) {
    runs.first[i + 1] = runs.first[i] + count(i);
    runs.most = std::max(runs.most, count(i));
  }
  return true;
}

hipError_t launch_attention_decode(const DecodeAttnParams& p, const RowMap& rm, const DecodeRuns& runs, float* part,
                                   int max_splits, hipStream_t s) {
  if (p.Hq % p.Hkv != 0 || p.page != kPage) return hipErrorInvalidValue;
  const int G = p.Hq / p.Hkv;
  if (G > 8 || (G & (G - 1)) != 0) return hipErrorInvalidValue;
  if (runs.most > max_splits) return hipErrorInvalidValue;
  const DecodeAttnScratch sc = decode_attn_scratch(rm.n_seqs, p.Hq, p.Hkv, p.d, max_splits);
  int* ctr = reinterpret_cast<int*>(part);
  float* po = part + sc.out_floats;
  float* pml = part + sc.ml_floats;
  const int grid = runs.first[rm.n_seqs] * p.Hkv;
  if (p.d == 128 && runs.wide) attn_decode_kernel<128, 4><<<grid, 256, 0, s>>>(p, rm, runs, po, pml, ctr);
  else if (p.d == 128) attn_decode_kernel<128, 2><<<grid, 128, 0, s>>>(p, rm, runs, po, pml, ctr);
  else if (p.d == 64 && runs.wide) attn_decode_kernel<64, 4><<<grid, 256, 0, s>>>(p, rm, runs, po, pml, ctr);
  else if (p.d == 64) attn_decode_kernel<64, 2><<<grid, 128, 0, s>>>(p, rm, runs, po, pml, ctr);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pallas
