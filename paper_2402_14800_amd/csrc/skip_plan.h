// The plan of a routed forward.  Host arithmetic only, without HIP, so that a program built on the CPU can check it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "moeprune.h"
#include "tile_plan.h"

namespace moep {

struct SkipPlan {
  int64_t T; int E, H, F;
  int ks;                // slots per token (2 for the top-2 rule, k for the generalised rule)
  int kept_experts;      // experts that tokens can be routed to
  int64_t max_slots;     // ks T
  bool may_skip = false; // a threshold above zero: any part of them can be left
  bool few;              // bf16, few rows per expert: gemm_few.hip, no operand is re-laid out
  int tile_rows;         // rows per tile of the map
  int64_t max_tiles;     // upper bound on M tiles over all experts
  size_t off_logits, off_slot_token, off_slot_scale, off_slot_dest, off_pos, off_counts, off_seg_end,
         off_tile_expert, off_tile_row0, off_order_up, off_order_down, off_h, off_xp, off_w13, off_w2, off_slot_out, total;
  bool packed;           // bf16: packed-operand GEMMs (tile order tables are built)
};
// kept_experts decides the path, not the size of the workspace
int plan_skip(int64_t T, int E, int H, int F, moep_dtype dt, int ks, int kept_experts, SkipPlan* p, bool with_slot_out = true);

// Whether the 256-row GEMM's gate/up or down launch of a routed forward loads its weights past the caches: no expert that was
// pruned away is read, however many the layer has.  us per call, all the layer's experts counted / the kept ones: 3 of 16 experts,
// H 2048, F 5632, 127 tokens 132 / 89, 4 of them (184 MB of gate/up) 137 / 126; 2 of 8, H 2048, F 8192, 85 tokens 137 / 95; 4 of 32,
// H 2048, F 2816, 120 tokens 90 / 68.
inline bool routed_weights_stream(const SkipPlan& p, bool gate_up) {
  return gate_up ? streams_weights(p.F, p.H, true, p.kept_experts) : streams_weights(p.H, p.F, false, p.kept_experts);
}

// Most tokens that the one-workgroup dispatch takes, one thread each, and most entries of the tile orders: there it is shorter
// than the two kernels it stands for.  In two / in one, us: Mixtral shape (E 8, H 4096, F 14336), top-2, T = 300 12.2 / 10.6,
// 777 13.0 / 11.2, 1000 13.0 / 12.1; top-4, 500 14.0 / 13.4, 600 14.2 / 15.0; E 32, H 384, F 4096, top-2, 500 14.3 / 13.5,
// 600 15.2 / 19.6, top-4, 200 18.1 / 14.7, 400 18.8 / 22.8; 3072 entries, 1000 tokens 14.7 / 18.2.  Up to 256 tokens it is shorter for
// every k: calls with H = F = 64, E 24, k 8, T = 129 37.3 / 33.9, E 32, k 16, T = 180 4 to 7 us less, k 6, T = 257 the same.
// Routing, slots, the map of tiles and their order in launches of their own took 19 to 27 us from 513 tokens on.
constexpr int DISPATCH_ONE_MAX = 1024, DISPATCH_ONE_ORDER_MAX = 2048, DISPATCH_ONE_ALWAYS = 256;
constexpr int dispatch_one_tokens(int E, int slots) {
  const int by_slots = 2 * DISPATCH_ONE_MAX / slots, most = (by_slots < DISPATCH_ONE_MAX ? by_slots : DISPATCH_ONE_MAX) >> (E > 16 ? 1 : 0);
  return most > DISPATCH_ONE_ALWAYS ? most : DISPATCH_ONE_ALWAYS;
}

}  // namespace moep
