// Model handle and the per-call plan of the prefill and decode sequences.
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "kernels.h"
#include "pallas.h"

struct pallas_model {
  pallas_model_config cfg;
  const void* embed;
  const void* final_norm;
  const void* lm_head;
  std::vector<pallas_layer_weights> layers;
};

namespace pallas {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Workspace carve-up for `tokens` rows (prefill: sum of prefix lengths;
// decode: number of sequences).
struct Workspace {
  size_t resid, h, qkv, q, o, act, rope, part, split, split_bytes, attn_split, attn_split_bytes;
  size_t gemv_part, gemv_part_bytes, gemv_ctr, ssq, shared;
  int gemv_ctr_count;
  int decode_splits;   // decode attention: splits per sequence its section holds
  size_t total;
};

// Decode positions are below this bound: as many splits as a sequence has, as
// long as a workgroup takes.
constexpr int kDecodeMaxPos = kDecodeSplitsPerSeq * kDecodeMaxRun;
static_assert(kDecodeMaxPos == 16384, "the decode position limit");

// Bytes of partial sums and arrival counters that a decode step of up to
// kGemvMaxRows rows needs (the largest of its five projections').
struct GemvNeed {
  size_t part_bytes = 0;
  int counters = 0;
};
inline GemvNeed gemv_need(const pallas_model_config& c) {
  const int QKV = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim, QD = c.n_q_heads * c.head_dim;
  const int proj[5][3] = {{kEpiBf16, QKV, c.hidden}, {kEpiAddF32, c.hidden, QD}, {kEpiSwiGLU, c.ffn, c.hidden},
                          {kEpiAddF32, c.hidden, c.ffn}, {kEpiF32, c.vocab, c.hidden}};
  GemvNeed need;
  for (const auto& p : proj) {
    const GemvPlan pl = gemv_plan(p[0], p[1], p[2]);
    need.part_bytes = std::max(need.part_bytes, pl.part_bytes());
    need.counters = std::max(need.counters, pl.counters());
  }
  return need;
}
// Sums of squares of up to kGemvMaxRows rows: one partial per 16 columns
// (GemvPlan, whole tiles of up to 64 columns).
inline size_t norm_bytes(const pallas_model_config& c) { return (size_t(c.hidden) / 16 + 4) * kGemvMaxRows * 4; }

inline Workspace workspace_layout(const pallas_model_config& c, int64_t tokens, int64_t seqs) {
  Workspace w;
  const int64_t qkv = int64_t(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  size_t at = 0;
  auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes, 256); return o; };
  w.resid = take(size_t(tokens) * c.hidden * 4);
  w.h = take(size_t(tokens) * c.hidden * 2);
  w.qkv = take(size_t(tokens) * qkv * 2);
  w.q = take(size_t(tokens) * c.n_q_heads * c.head_dim * 2);
  w.o = take(size_t(tokens) * c.n_q_heads * c.head_dim * 2);
  w.act = take(size_t(tokens) * c.ffn * 2);
  w.rope = take(size_t(tokens) * (c.head_dim / 2) * 8);  // (cos, sin) per row and pair
  w.shared = take(size_t(seqs) * 4);                     // decode: a flag per row
  w.decode_splits = kDecodeSplitsPerSeq;
  w.part = take(decode_attn_scratch(int(seqs), c.n_q_heads, c.n_kv_heads, c.head_dim, w.decode_splits).floats * 4);
  w.ssq = take(norm_bytes(c));   // decode: sums of squares
  // Split-K partial sums of the projections of up to 256 rows.
  {
    const int rows = static_cast<int>(tokens < 256 ? tokens : 256);
    const int H = c.hidden, QD = c.n_q_heads * c.head_dim, KVD = 2 * c.n_kv_heads * c.head_dim;
    size_t b = gemm_split_bytes(kEpiBf16, rows, static_cast<int>(qkv), H);
    b = std::max(b, gemm_split_bytes(kEpiBf16, rows, KVD, H));
    b = std::max(b, gemm_split_bytes(kEpiAddF32, rows, H, QD));
    b = std::max(b, gemm_split_bytes(kEpiSwiGLU, rows, c.ffn, H));
    b = std::max(b, gemm_split_bytes(kEpiAddF32, rows, H, c.ffn));
    b = std::max(b, gemm_split_bytes(kEpiF32, rows, c.vocab, H));
    w.split_bytes = b;
    w.split = take(b);
  }
  // Split records of prefill attention over up to 256 rows.
  w.attn_split_bytes = attn_prefill_split_bytes(static_cast<int>(tokens < 256 ? tokens : 256),
                                                c.n_q_heads, c.head_dim);
  w.attn_split = take(w.attn_split_bytes);
  // Decode projections split over K: partial sums and arrival counters.
  {
    const GemvNeed need = gemv_need(c);
    w.gemv_part_bytes = need.part_bytes;
    w.gemv_part = take(need.part_bytes);
    w.gemv_ctr_count = need.counters;
    w.gemv_ctr = take(size_t(need.counters) * 4);
  }
  w.total = at;
  return w;
}

// The documented scratch need of pallas_decode_step_static, which decides
// what it accepts: the step's activations, one record per 64 keys and query
// head, and partial sums and counters of the projections of fewer than 512
// 16-row tiles.  It is what the first decode kernels used and is kept so that
// the same calls are accepted; the layout itself is decode_layout.
inline size_t static_decode_need(const pallas_model_config& c, int seqs, int max_pos) {
  const int64_t QKV = int64_t(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  const int64_t QD = int64_t(c.n_q_heads) * c.head_dim;
  size_t at = 0;
  auto take = [&](size_t bytes) { at = align_up(at + bytes, 256); };
  take(size_t(seqs) * c.hidden * 4);
  take(size_t(seqs) * c.hidden * 2);
  take(size_t(seqs) * QKV * 2);
  take(size_t(seqs) * QD * 2);
  take(size_t(seqs) * QD * 2);
  take(size_t(seqs) * c.ffn * 2);
  take(size_t(seqs) * (c.head_dim / 2) * 8);
  take(size_t(seqs) * c.n_q_heads * (max_pos / 64 + 1) * (c.head_dim + 2) * 4);
  auto splits = [](int64_t N, int64_t K, int resident) {
    const int64_t tiles = (N + 15) / 16;
    int best = 1;
    if (tiles >= 512) return best;
    auto even = [&](int s) { return double(tiles) * s / 256.0 / std::ceil(double(tiles) * s / 256.0); };
    for (int s = 2; s <= 8 && K / (s * 256) >= 4 && tiles * s <= resident; ++s)
      if (even(s) > even(best) + 0.05) best = s;
    return best;
  };
  const int64_t proj[5][4] = {{QKV, c.hidden, 1024, QKV}, {c.hidden, QD, 1024, c.hidden},
                              {c.ffn, c.hidden, 512, 2 * int64_t(c.ffn)}, {c.hidden, c.ffn, 1024, c.hidden},
                              {c.vocab, c.hidden, 1024, c.vocab}};
  size_t part = 0, tiles = 0;
  for (const auto& p : proj) {
    const int s = splits(p[0], p[1], int(p[2]));
    if (s == 1) continue;
    part = std::max(part, size_t(s) * seqs * p[3] * 4);
    tiles = std::max(tiles, size_t((p[0] + 15) / 16));
  }
  take(part);
  take(tiles * 4);
  return at;
}

// The layout a decode step of `seqs` <= 8 sequences runs in without a
// workspace, with positions up to `max_pos` (the same plans and kernels as in a
// full workspace).
inline Workspace decode_layout(const pallas_model_config& c, int seqs, int max_pos) {
  Workspace w{};
  const int64_t QKV = int64_t(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  const int64_t QD = int64_t(c.n_q_heads) * c.head_dim;
  size_t at = 0;
  auto take = [&](size_t bytes) { size_t o = at; at = align_up(at + bytes, 256); return o; };
  w.resid = take(size_t(seqs) * c.hidden * 4);
  w.h = take(size_t(seqs) * c.hidden * 2);
  w.qkv = take(size_t(seqs) * QKV * 2);
  w.o = take(size_t(seqs) * QD * 2);
  w.act = take(size_t(seqs) * c.ffn * 2);
  w.rope = take(size_t(seqs) * (c.head_dim / 2) * 8);
  w.shared = take(size_t(seqs) * 4);
  w.decode_splits = std::min(max_pos / kDecodeMinSplit + 1, kDecodeSplitsPerSeq);
  w.part = take(decode_attn_scratch(seqs, c.n_q_heads, c.n_kv_heads, c.head_dim, w.decode_splits).floats * 4);
  w.ssq = take(norm_bytes(c));
  const GemvNeed need = gemv_need(c);
  w.gemv_part_bytes = need.part_bytes;
  w.gemv_part = take(need.part_bytes);
  w.gemv_ctr_count = need.counters;
  w.gemv_ctr = take(size_t(need.counters) * 4);
  w.total = at;
  return w;
}

inline size_t workspace_bytes(const pallas_model_config& c, int32_t max_tokens, int32_t max_seqs) {
  return workspace_layout(c, max_tokens, max_seqs).total;
}

}  // namespace pallas
