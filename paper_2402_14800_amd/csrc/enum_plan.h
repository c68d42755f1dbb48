// The plan of a subset enumeration.  Host arithmetic only, without HIP, so that a program built on the CPU can check it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace moep {

struct EnumPlan {
  int64_t T; int E, H, k, r;
  int kk;            // min(k, r): experts per token in the pruned layer
  int n_act;         // min(E, kk + E - r): rank positions that can be selected
  int64_t n_sub;     // C(E, r)
  int rec_floats;    // floats per token record
  int tok_tile;      // tokens per scoring block
  int64_t n_tok_tiles;
  bool use_lut;      // many subsets, few selections per token: score through per-token selection tables
  int n_combo;       // C(n_act, kk): selections per token
  int fused_threads; // up to 16 experts: tables and look-ups in one kernel, its workgroup (0: not taken),
  int fused_spl;     //   subsets per lane,
  int fused_tg;      //   tokens per barrier
  size_t fused_lds;  //   and dynamic LDS
  // workspace carving (byte offsets)
  size_t off_gram, off_rec, off_masks, off_partial, off_partial_cnt, off_qtab, off_sel, off_selbits, off_nib, total;
};
int plan_enumerate(int64_t T, int E, int H, int k, int r, EnumPlan* p);

// The Gram pass writes the records of up to RECORD_SETS values of r itself, and the Gram matrices never go to memory, where
// records_by_gram_pass says so; where it puts each r's records, partial sums and counts (byte offsets in the workspace).
constexpr int RECORD_SETS = 4;
struct RecordPlan { size_t rec[RECORD_SETS], partial[RECORD_SETS], cnt[RECORD_SETS]; };

// A wavefront takes 4, 2 or 1 tokens (a tile) of `rows` rows each, up to 16 in all; their records cost it a few us of latency, which
// the memory traffic of the wavefronts beside it hides only where a tile is long.  What that saves are launches of 5 to 10 us and,
// the longer the records, some time per token; from the rank-limited pass also Gram matrices of E x E entries for `rows` experts.
// So: batches of few tiles, and tiles of 32 KB (ranked 16, not mostly padding), in fp32, where the products take longer, of twice that
// and not mostly padding.  us per call, Gram matrices in memory / records, bf16: E 16, k 2, r 14, H 256, T = 4000 40 / 35, 8000 48 / 50, 65536 171 /
// 252; H 512 (16 KB), T = 65536 236 / 267, H 1024 (32 KB) 429 / 393; k 8, r 15, H 64, T = 8000 58 / 51, 16000 73 / 84; E 8, r 6 and
// 4, H 64, T = 16000 61 / 52, 65536 129 / 152; ranked, E 16, k 4, r 12, 8 rows, H 512 (16 KB), T = 40000 171 / 149.  fp32, E 8, r 6
// and 4, H 1024 (64 KB), T = 65536 458 / 441; E 9 (7 rows of padding), H 2048, T = 32000 469 / 507.
// Ranked, from where they are even, H 64 to 320: 2 of 2 experts about T = 12000 (4 tokens to a tile), 4 of 5 15000, 6 of 6 10000 (2), 8 of 8
// 14000, 8 of 16, r 14, 20000, 16 of 16, r 12, 11000 (1), 12 of 12, r 6, 15000.
constexpr int64_t RECORD_TILES = 2304;                     // times the sum over the r of record_weight
constexpr int64_t record_tiles_ranked(int tokens) { return tokens == 4 ? 1536 : tokens == 2 ? 2560 : 3584; }
constexpr int64_t RECORD_TILE_BYTES = 32 * 1024;
constexpr int record_weight(int n_act) { return n_act <= 4 ? 2 : n_act <= 8 ? 3 : 4; }
constexpr int record_tile_tokens(int rows) { return rows <= 4 ? 4 : rows <= 8 ? 2 : 1; }
constexpr bool records_pay(int64_t T, int rows, int H, bool f32, bool ranked, int weights) {
  const int tokens = record_tile_tokens(rows);
  const int64_t bytes = (int64_t)tokens * rows * H * (f32 ? 4 : 2);
  return (T + tokens - 1) / tokens <= (ranked ? record_tiles_ranked(tokens) : RECORD_TILES) * weights ||
         (bytes >= RECORD_TILE_BYTES * (f32 ? 2 : 1) / (ranked ? 2 : 1) && (tokens * rows >= 12 || !(f32 || ranked)));
}
// `plans`: n of one batch; n_rank: rows of Y per token, 0: all E; ws_bytes: of the workspace, which is sized for Gram matrices and
// one r.
bool records_by_gram_pass(const EnumPlan* const* plans, int n, int n_rank, bool f32, size_t ws_bytes, RecordPlan* out);

}  // namespace moep
