// Internal launch interface between the C ABI (pallas_api.hip) and the
// kernels.  Every launcher enqueues on `s` and returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pallas {

// ----------------------------------------------------------------- KV copies
struct PoolGeom {
  char* base;         // bf16 [L][2][num_pages][page][Hkv][d]
  int32_t num_pages;
  int32_t page;
  int32_t lk;         // 2 * L: (layer, K|V) planes
  int32_t row_bytes;  // Hkv * d * 2, a multiple of 16
};

constexpr int kCopyMaxChunks = 128;   // chunks per copy launch
constexpr int kCopyTokens = 16;       // tokens per work unit

struct CopyChunk {
  int32_t start;       // first logical position
  int32_t count;       // positions
  uint64_t offset;     // byte offset of [2L][count][row] in the arena
};
struct CopyBatch {
  int32_t n;
  int32_t unit_prefix[kCopyMaxChunks + 1];  // work units before chunk j
  CopyChunk c[kCopyMaxChunks];
};

// Pack (pool -> arena) or assemble (arena -> pool) of up to kCopyMaxChunks
// chunks through one block table.
hipError_t launch_kv_copy(bool pack, const PoolGeom& pool, const int32_t* bt, char* arena,
                          const CopyBatch& b, int32_t* d_err, hipStream_t s);

}  // namespace pallas

namespace pallas {

// ---------------------------------------------------------------- GEMM
enum GemmEpi : int {
  kEpiBf16 = 0,    // C bf16 [M][ldc] = A B^T
  kEpiAddF32 = 1,  // C f32 [M][ldc] += A B^T (residual add)
  kEpiSwiGLU = 2,  // C bf16 [M][ldc] = silu(A Bg^T) * (A Bu^T); B rows [0,N) gate, [N,2N) up
  kEpiF32 = 3,     // C f32 [M][ldc] = A B^T (decode: up to 64 rows)
};

struct GemmParams {
  const uint16_t* A;
  const uint16_t* B;
  void* C;
  int M, N, K;
  int lda, ldb, ldc;
  int tiles_m, tiles_n, total_tiles, tiles_per_xcd, group_m;
  int tail_half;        // full tiles per XCD run split into two half-width tiles (tail kernel)
  int ksplit;           // K-range splits per tile (1: none)
  float* part;          // split partial sums [ksplit][M][part_ld] (ksplit > 1)
  int part_ld;          // B rows: N, or 2N for the gate|up product
  uint32_t a_bytes, b_bytes;
  // Clock sampling (profiling only, else null): each workgroup adds its
  // shader-clock cycles, wall-clock ticks and 1 to clk[0], clk[1], clk[2].
  unsigned long long* clk;
};

// Output-column tiles for tiles of bn B rows (gate|up: bn/2 gate + bn/2
// up rows, so bn/2 output columns per tile).
inline int gemm_tiles_n(int epi, int N, int bn = 256) {
  const int cols = epi == kEpiSwiGLU ? bn / 2 : bn;
  return (N + cols - 1) / cols;
}
// Tile shape (output rows bm x B rows bn) of a launch without a K split.
// Every shape runs the same MFMA over the same K order, so the choice never
// changes an output bit.  A launch takes rounds of one workgroup per CU,
// dealt to the 8 XCDs' 32 CUs each; its time is modelled as rounds x tile
// area / the shape's FLOP rate per CU relative to 256 x 256, measured at
// the large and mid shapes (a 256 x 256 launch whose last round keeps at
// most half the CUs busy runs that round as half-width tiles, at
// 0.5 / 0.77 of a round).  The 192-row shapes fit row counts such as
// 1536 = 8 x 192 (the mid model: Q|K|V 144 tiles of 256 x 256 but 256 of
// 192 x 192; O and down 96 but 256 of 192 x 128).  A shape replaces the
// best so far only when modelled at least 1% cheaper, so near-ties keep
// the earlier (larger) tile: at the mid model's gate|up, 1536 rows, the
// split-tail 256 x 256 launch and 192 x 256 model within 0.1% of each
// other, and the 256 x 256 one measured 248-250 against 253 us.  The
// 128-row shapes spread a few hundred rows over more CUs: 500 rows of the mid
// model's O 40.9 (192 x 128) -> 29.6 us (128 x 64), its down 118 -> 80; 320
// rows of the large model's O 74 -> 44 us, its down 248 -> 135.  128 x 96 is
// for launches that 128 x 64 would run in two rounds: 500 rows of the large
// model's O 69 (128 x 128) -> 63 us, its down 232 -> 201; 640 rows of the mid
// model's O 39 -> 35, its down 114 -> 102.
struct GemmTile {
  int bm, bn;
};
inline GemmTile gemm_tile(int epi, int M, int N) {
  struct Cand {
    int bm, bn, rate;   // rate: FLOP rate per CU, percent of 256 x 256
  };
  static const Cand cands[] = {{256, 256, 100}, {256, 128, 77}, {192, 256, 85}, {192, 192, 80}, {192, 128, 70},
                               {128, 128, 49}, {128, 96, 44}, {128, 64, 38}};
  GemmTile best{256, 256};
  double best_cost = 0;
  for (const Cand& c : cands) {
    // gate|up: blocks pair up (no 96 or 192-wide tiles), and its many columns
    // never leave so few tiles that the 128-row shapes paid
    if (epi == kEpiSwiGLU && (c.bn == 192 || c.bm == 128)) continue;
    const int tiles = ((M + c.bm - 1) / c.bm) * gemm_tiles_n(epi, N, c.bn);
    const int per_xcd = (tiles + 7) / 8, rounds = (per_xcd + 31) / 32;
    double r = rounds;
    if (c.bm == 256 && c.bn == 256 && rounds > 1 && per_xcd - 32 * (rounds - 1) <= 16) r = rounds - 1 + 0.5 / 0.77;
    const double cost = r * c.bm * c.bn / c.rate;
    if (best_cost == 0 || cost < 0.99 * best_cost) {
      best = {c.bm, c.bn};
      best_cost = cost;
    }
  }
  return best;
}

// Launches of at most kGemmFewRows rows take one M tile, the shortest that
// covers them, with columns of 128 B rows, or of 256 where the 128-wide tiles
// need another round of the 256 CUs that the 256-wide ones do not (a 256-wide
// round takes about 1.75 times as long): gate|up of the large model at 128
// rows 129 -> 110 us.
constexpr int kGemmFewRows = 256;
inline GemmTile gemm_tile_few(int epi, int M, int N) {
  auto rounds = [&](int bn) { return (gemm_tiles_n(epi, N, bn) + 255) / 256; };
  const int bn = rounds(256) * 1.75 < rounds(128) ? 256 : 128;
  if (M <= 64 && bn == 128) return {64, 128};
  return {M <= 128 ? 128 : M <= 192 ? 192 : 256, bn};
}
// Which of the two tile rules a launch takes.  Without a K split (K below 2048,
// or many columns), more than 64 rows are one M tile only where gemm_tile, too,
// takes one, of at least 128 columns, and the columns fill a quarter of the
// CUs.  Fewer run faster as gemm_tile's, in narrower tiles or two M tiles, and
// with their few weights cached: the tiny model's prefill of 192 rows takes 86
// against 121 us, one of hidden 1536 and ffn 8960 198 against 273 at 256 rows.
// At 180 rows and 32, 64, 96 and 140 tiles of gate|up, three layers take 161,
// 176, 186 and 192 us that way, 173, 174, 177 and 181 this way; 288 tiles of
// 128 in 256 rows 1089 against 1022.
inline bool gemm_few_rows(int epi, int M, int N, int ksplit) {
  if (M > kGemmFewRows || M <= 64 || ksplit > 1) return M <= kGemmFewRows;
  const GemmTile t = gemm_tile(epi, M, N);
  return t.bm >= M && t.bn >= 128 && gemm_tiles_n(epi, N, 128) >= 64;
}

// K-range splits per tile.  Only launches of at most 256 rows split (their
// few tiles would leave most of the 256 CUs idle): 128-wide tiles times
// splits fill at most 256 workgroups, and each split keeps at least 16 K-steps
// of 64 (fewer splits, larger tiles and less partial-sum traffic than with
// 256 x 256 tiles: at 256 rows Q|K|V / O / down of the large model 52 / 47 /
// 94 -> 41 / 36 / 80 us, of the mid one 37 / 31 / 52 -> 27 / 21 / 41; at 64
// rows 39 / 34 / 72 -> 26 / 23 / 54).  The factor depends on N and K alone
// within M <= 256, and is 1 above, so a row's arithmetic is the same in
// prefills of any two lengths on the same side of 256 rows.
inline int gemm_ksplit(int epi, int M, int N, int K) {
  if (M > kGemmFewRows || N % 4 != 0) return 1;
  int s = 256 / gemm_tiles_n(epi, N, 128);
  if (s > K / 1024) s = K / 1024;
  if (s > 16) s = 16;
  return s < 1 ? 1 : s;
}
// Bytes of float32 partial sums a split GEMM needs (0 when it does not split).
inline size_t gemm_split_bytes(int epi, int M, int N, int K) {
  const int s = gemm_ksplit(epi, M, N, K);
  return s > 1 ? size_t(s) * M * (epi == kEpiSwiGLU ? 2 * size_t(N) : size_t(N)) * 4 : 0;
}

// A bf16 [M][lda] (K columns used), B bf16 [rows][ldb]; K a multiple of 8;
// A and B 16-byte aligned; M*lda*2 and rows*ldb*2 below 2 GiB.  When the
// GEMM splits K (gemm_ksplit > 1), `part` (16-byte aligned, at least
// gemm_split_bytes) receives the partial sums and a second kernel reduces
// them into C; ldc must then be a multiple of 4.
// `norm` (kEpiAddF32): where gemm_fuses_norm, the RMSNorm of the new C, h
// [M][N] = bf16(C / rms(C) gain), is written by the reduction.
struct GemmNorm {
  const uint16_t* gain;
  uint16_t* h;
  float eps;
};
inline bool gemm_fuses_norm(int epi, int M, int N, int K) {
  return epi == kEpiAddF32 && N <= 8192 && gemm_ksplit(epi, M, N, K) > 1;
}
hipError_t launch_gemm(int epi, const uint16_t* A, int lda, const uint16_t* B, int ldb, void* C,
                       int ldc, int M, int N, int K, float* part, size_t part_bytes, hipStream_t s,
                       unsigned long long* clk = nullptr, const GemmNorm* norm = nullptr);

}  // namespace pallas

namespace pallas {

// ------------------------------------------------------------ row metadata
constexpr int kMaxSeqs = 64;
constexpr int kMaxPrefillLen = 32768;  // tokens per sequence in one prefill call

// Rows [cu[s], cu[s+1]) belong to sequence s and sit at positions
// base_pos[s] + (row - cu[s]); sequence s uses block-table row s.
struct RowMap {
  int32_t n_seqs;
  int32_t cu[kMaxSeqs + 1];
  int32_t base_pos[kMaxSeqs];
};

__host__ __device__ inline int row_seq(const RowMap& rm, int row) {
  int s = 0;
  while (s + 1 < rm.n_seqs && rm.cu[s + 1] <= row) ++s;
  return s;
}

// ------------------------------------------------------------ norms / embed
// r[t] = float(E[ids[t]]); h[t] = bf16(rmsnorm(r[t]) * g); tab[t][i] = (cos,
// sin)(pos(t) * theta^(-2i/d)), evaluated in double; the spans are cleared
// (by the kernel, so a captured graph holds no memset).  `shared` (decode of
// several rows; flag null: none): flag[i] = 1 where row i may attend to a slot
// that another row of the call writes, else 0.
struct ClearSpan {
  int32_t* p;
  int n;
};
struct SharedSlots {
  const int32_t* bt;
  int max_pages, num_pages, page;
  int32_t* flag;
};
hipError_t launch_embed_rmsnorm(const int32_t* ids, const uint16_t* embed, const uint16_t* gain,
                                float* r, uint16_t* h, int rows, int H, float eps, int vocab,
                                int32_t* err, const RowMap& rm, int d, float theta, float* tab,
                                ClearSpan a, ClearSpan b, const SharedSlots& shared, hipStream_t s);
// h[t] = bf16(rmsnorm(r[t]) * g)
hipError_t launch_rmsnorm(const float* r, const uint16_t* gain, uint16_t* h, int rows, int H,
                          float eps, hipStream_t s);

// ------------------------------------------------------------ QKV epilogue
struct QkvParams {
  const uint16_t* qkv;     // [rows][qkv_ld]: Q heads, K heads, V heads (or K, V only)
  int qkv_ld;
  int kv_only;             // 1: qkv holds only the K and V heads
  const uint16_t* q_gain;  // [d] or null
  const uint16_t* k_gain;  // [d] or null
  const float* rope;       // [rows][d/2][2]
  uint16_t* q_out;         // [rows][Hq][d] (unused when kv_only)
  uint16_t* k_plane;       // pool K plane of this layer: [P][page][Hkv][d]
  uint16_t* v_plane;       // pool V plane
  const int32_t* bt;       // [n_seqs][max_pages]
  int max_pages, num_pages, page;
  int Hq, Hkv, d;
  float eps;
  int qk_norm;
  int32_t* err;
};
hipError_t launch_qkv_rope(const QkvParams& p, const RowMap& rm, int rows, hipStream_t s);

// ------------------------------------------------------------ attention
struct AttnParams {
  const uint16_t* q;       // [rows][Hq][d]
  const uint16_t* k_plane; // [P][page][Hkv][d]
  const uint16_t* v_plane;
  const int32_t* bt;
  int max_pages, num_pages, page;
  int64_t plane_bytes;     // bytes of one K (or V) plane: num_pages * page * Hkv * d * 2
  uint16_t* o;             // [rows][Hq * d]
  int Hq, Hkv, d;
  float scale_log2;        // log2(e) / sqrt(d)
};
// Key-range splits of prefill attention.  Only calls of at most 256 rows
// split (as the GEMMs, so longer prefills keep identical bytes per row),
// and only when their (query block, KV head) workgroups are too few to fill
// the chip: up to 8 splits of at least 2 key tiles of 64, as many as run at
// once (two workgroups per CU: a 256-token chunk at position 2744 of the large
// model, 144 workgroups, took 55 us in 576 and 47 in 432).
inline int attn_prefill_splits(int rows, int workgroups, int max_tiles) {
  if (rows > 256 || workgroups >= 256) return 1;
  int s = 512 / workgroups;
  if (s > 8) s = 8;
  if (s > max_tiles / 2) s = max_tiles / 2;
  if (s < 1) return 1;
  const int per = (max_tiles + s - 1) / s;
  return (max_tiles + per - 1) / per;
}
// Bytes of split records the workspace holds for up to `rows` rows:
// [rows][Hq][8][d + 4] floats.
inline size_t attn_prefill_split_bytes(int rows, int Hq, int d) {
  return size_t(rows < 256 ? rows : 256) * Hq * 8 * (d + 4) * 4;
}
// Causal prefill attention: row t of sequence s is position base_pos[s] +
// (t - cu[s]) and attends to keys of its own table at positions <= its
// own, [0, base_pos[s]) written by earlier calls.  `part` (split records,
// attn_prefill_split_bytes) is used when the call splits its key ranges.
hipError_t launch_attention_prefill(const AttnParams& p, const RowMap& rm, float* part, size_t part_bytes,
                                    hipStream_t s);
// Decode attention and what precedes it: QK-norm and rotary of the row's Q and
// K, the store of its K and V into slot base_pos[s], then attention over keys
// [0, base_pos[s]] through the table (rows on pages outside the pool masked).
struct DecodeAttnParams {
  const uint16_t* qkv;     // [rows][qkv_ld]: Q heads, K heads, V heads
  int qkv_ld;
  const uint16_t* q_gain;  // [d] or null
  const uint16_t* k_gain;  // [d] or null
  const float* rope;       // [rows][d/2][2]
  float eps;
  int qk_norm;
  uint16_t* k_plane;       // [P][page][Hkv][d]
  uint16_t* v_plane;
  const int32_t* bt;
  int max_pages, num_pages, page;
  uint16_t* o;             // [rows][Hq * d]
  int Hq, Hkv, d;
  float scale_log2;        // log2(e) / sqrt(d)
  const int32_t* shared;   // [rows] of the call's start (SharedSlots); read when there are several rows
  int32_t* err;
};
// Keys per split of a sequence at position n, from n alone: 128, and as many
// more as keep a sequence at 16 splits.  One sequence (large layer, us): 1000
// keys 9.9 in 128-key splits, 11.4 in 256, 13.8 in 512; 4000 keys 12.0 in 16
// splits, 14.3 in 8; 8000 keys 15.2 in 16, 20 in 8; more than 16 cost more in
// the merge than they save (4000 keys in 32: 17.5, before in 16 14.1).
constexpr int kDecodeMinSplit = 128;
constexpr int kDecodeSplitsPerSeq = 16;
constexpr int kDecodeMaxRun = 1024;     // keys of a workgroup: its table entries, one per lane
constexpr int kDecodeMaxRunSplits = 4;  // its merges in progress are held in registers
__host__ __device__ inline int decode_split_keys(int n) {
  return (n / kDecodeSplitsPerSeq + kDecodeMinSplit) / kDecodeMinSplit * kDecodeMinSplit;
}
// The section of decode attention for up to max_splits splits per sequence:
// arrival counters (zero on entry, left zero), outputs [n_seqs][Hkv][run][G]
// [d], then maxima and sums.  With one split nothing is used.
struct DecodeAttnScratch {
  int counters;            // ints to clear at the start of the section
  size_t out_floats, ml_floats, floats;
};
inline DecodeAttnScratch decode_attn_scratch(int n_seqs, int Hq, int Hkv, int d, int max_splits) {
  DecodeAttnScratch s;
  s.counters = max_splits > 1 ? n_seqs * Hkv : 0;
  s.out_floats = (size_t(n_seqs) * Hkv + 63) / 64 * 64;
  s.ml_floats = s.out_floats + size_t(n_seqs) * Hq * max_splits * d;
  s.floats = max_splits > 1 ? s.ml_floats + size_t(n_seqs) * Hq * max_splits * 2 : 0;
  return s;
}
// Work of a call: sequence s has runs [first[s], first[s + 1]) of per_run[s]
// splits each (a power of two), one workgroup per run and KV head.
struct DecodeRuns {
  int32_t wide;                     // four waves per workgroup, else two
  int32_t most;                     // the largest run count of a sequence
  int32_t first[kMaxSeqs + 1];
  int32_t per_run[kMaxSeqs];
};
// False where a position is outside what the kernel takes.
bool plan_decode_runs(const RowMap& rm, int Hkv, DecodeRuns& runs);
hipError_t launch_attention_decode(const DecodeAttnParams& p, const RowMap& rm, const DecodeRuns& runs, float* part,
                                   int max_splits, hipStream_t s);

// ------------------------------------------------------------ skinny GEMM
// C[m][n] (op) A[m] . B[n] for m < M <= 8 rows (gemv.hip); epilogues as
// launch_gemm.
constexpr int kGemvMaxSplit = 8;
constexpr int kGemvMaxRows = 8;

// How a projection runs: workgroups of 4 waves, each a tile of tn blocks of
// 16 weight rows over 1 / S of K.
struct GemvPlan {
  int tn, S;
  int tiles;
  size_t part_bytes() const { return S > 1 ? size_t(tiles) * S * tn * 1024 : 0; }
  int counters() const { return S > 1 ? tiles : 0; }
  // Sum-of-squares partials of the residual epilogue, each kGemvMaxRows floats.
  int norm_parts() const { return tiles * tn; }
};
// The plan of least modelled time, from the shape alone (so a row's arithmetic
// does not depend on the rows beside it; X, a small part of the loads, is not
// counted).  A CU holds r workgroups (their LDS stages decide), and a full
// round of 256 r of them takes K / S u r + c0: u = the time 256 CUs need for
// one k of tn blocks at 5.5 TB/s, c0 = 3 us of start and epilogue.  A split
// adds 1 us + 0.3 us per part (count, partial sums) and the partials' traffic.
//   It ranks plans and predicts no times: modelled against measured (us, tn /
// S), Q|K|V of the mid model 1 / 2 14.1, 11.8; 2 / 1 15.2, 12.7; 2 / 4 15.1,
// 14.2 (8 rows); of the large one 4 / 3 26.2, 19.7; 1 / 1 25.9, 20.2; large O
// 2 / 3 21.7, 17.6; down 2 / 3 56.2, 43.2; 1 / 3 56.2, 45.  Equal ones keep the
// narrower tile: at the large down and Q|K|V that is 4% and 3% off the best.
inline GemvPlan gemv_plan(int epi, int N, int K) {
  GemvPlan best{};
  const int64_t rows = epi == kEpiSwiGLU ? 2 * int64_t(N) : N;
  double best_t = 0;
  for (int tn = 1; tn <= 4; tn *= 2) {
    if (tn == 1 && epi == kEpiSwiGLU) continue;
    const int stages = tn == 1 ? 3 : 2;
    const int lds = 4 * stages * (2 * tn + 1) * 1088 + 1024;   // 8-row blocks of 68 x 16 bytes
    const int resident = 160 * 1024 / lds;
    const int per = epi == kEpiSwiGLU ? tn * 8 : tn * 16;       // output columns per tile
    const int tiles = (N + per - 1) / per;
    const double u = tn * 32.0 * 256 / 5.5e6;                   // us per k and workgroup of a CU
    for (int S = 1; S <= kGemvMaxSplit; ++S) {
      const GemvPlan pl{tn, S, tiles};
      const int64_t wgs = int64_t(tiles) * S;
      if (S > 1 && (K / (S * 256) < 4 || wgs > 256 * resident)) break;
      const double full = double(wgs / (256 * resident)), rest = double(wgs % (256 * resident));
      double t = full * (double(K) / S * u * resident + 3);
      if (rest > 0) t += double(K) / S * u * double((int(rest) + 255) / 256) + 3;
      if (S > 1) t += 1 + 0.3 * S + 2.0 * S * rows * 64 / 4e6;
      if (best_t == 0 || t < best_t * 0.999) {
        best = pl;
        best_t = t;
      }
    }
  }
  return best;
}

struct GemvScratch {
  float* part;
  size_t part_bytes;
  int* ctr;         // zero on entry, left zero
  int ctr_count;
};
// The RMSNorm before and after a projection.  In: A holds x g, and row m's
// output is scaled by (sum of ssq_in[0..parts_in)[m] / K + eps)^(-1/2)
// (ssq_in null: no scale).  Out (kEpiAddF32 only, gain_out not null): h_out =
// bf16(C gain_out), laid out as C, and the sums of squares of C's rows in
// ssq_out[norm_parts()][kGemvMaxRows] of the plan.
struct GemvNorm {
  const float* ssq_in;
  int parts_in;
  float eps;
  const uint16_t* gain_out;
  uint16_t* h_out;
  float* ssq_out;
};
hipError_t launch_gemv(int epi, const uint16_t* A, int lda, const uint16_t* B, int ldb, void* C, int ldc, int M, int N,
                       int K, const GemvScratch& sc, const GemvNorm& nrm, hipStream_t s);

}  // namespace pallas
