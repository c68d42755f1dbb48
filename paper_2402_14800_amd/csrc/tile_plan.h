// How the 256-row GEMM's launches are cut into tiles.  Plain arithmetic, without HIP: the dispatch kernels call it, and so does a
// program built on the CPU that checks it.
#pragma once

#include <stdint.h>

namespace moep {

// Whether a launch of `tiles` full-width tiles is shorter with twice as many of half the width, on 256 compute units: while
// they still fit one round.  Forward of 777 tokens at the Mixtral shape (128 tiles in its down projection) 764 -> 716 us,
// dense pass of 64 tokens 798 -> 739 us; with 896 gate/up tiles taken as 7 half rounds for 4 the former was 790 us, and 160
// tiles as two half rounds for one cost 445 -> 507 us (E 16, H 2048, F 5632, top-4, 1001 tokens).
constexpr bool half_width_pays(int64_t tiles) { return tiles <= 128; }

// Full-width tiles at the end of a routed launch of `tiles` that are walked as two of half the width each: those of a last round
// that half of the compute units would otherwise sit out.  us per call, without / with: E 16, H 2304, F 2368, T = 3133
// (2.4 rounds) 339 / 315; E 8, H 1920, F 7168, top-4, T = 2240 778 / 723; E 8, H 4096, F 14336, T = 969 899 / 882.  Below
// TAIL_MIN_K what a tile saves goes into the second ring's fill (E 4, H 576, F 4032, top-4, T = 544 92 / 97; E 8, H 896, F 1984,
// T = 2427 109 / 111).  Not with tiles of up to 128 rows (row_groups 4), whose steps are the load of the weights: E 8, H 4096,
// F 14336, T = 262 581 / 606, E 16, H 2048, F 5632, T = 900 275 / 286.  n_full, n_half: tiles of either width along N; the launch's
// table has room for n_half per M tile, which is enough for both kinds where n_half > n_full.
constexpr int TAIL_MIN_K = 1024;
constexpr int64_t tail_tiles(int64_t tiles, int n_full, int n_half, int k, int row_groups) {
  return tiles > 256 && n_half > n_full && k >= TAIL_MIN_K && row_groups > 4 && half_width_pays(tiles & 255) ? tiles & 255 : 0;
}

// Weights of a launch from which they are loaded past the caches.  `experts`: the ones that can have rows.
constexpr double STREAM_BYTES = 192e6;
constexpr bool streams_weights(int N, int K, bool gate_up, int experts) {
  return (double)N * K * 2.0 * (gate_up ? 2.0 : 1.0) * experts > STREAM_BYTES;
}

// Rows per tile of a routed launch: 256, or SHORT_TILE_ROWS where the call's two launches are shorter with that.  What they
// cost is the rounds of 256 tiles (compute units) that they take, each as many steps as its K is deep and the epilogue: about
// 4 steps of 32 for the SwiGLU one, 24 for the row-scaled one.  A 192-row tile costs 13/16 of a 256-row one (6/8 of the products,
// but the same weights), and a launch of half-width tiles, which fits one round, 10/16 of a round.  256 / 192 rows, us per call, no
// token skipped: E 16, H 2048, F 5632, top-4, T = 1200 492 / 435, T = 1500 (a 257th tile in the down projection) 495 / 527; E 8, H 1024,
// F 3584, T = 1500 126 / 120; Mixtral shape, T = 2000 1368 / 1339, T = 777 with some expert beyond 192 rows 762 / 875.  The epilogues
// matter where K is a few hundred (E 32, H 3136, F 128, T = 3006, three rounds of 4 steps for two: 122 / 141; E 32, H 1664, F 64, top-4,
// T = 1591 85 / 88).
// The price counts whole rounds: neither a last round in half tiles (above) nor the row-scaled epilogue's loads, which have come
// together since the 24 steps were fitted, are in it.  Where they would turn the choice, both heights were timed: Mixtral shape, T = 900
// 755 / 944, E 4, H 1408, F 4096, top-4, T = 4647 598 / 598, E 32, H 2176, F 960, top-4, T = 4206 372 / 338: the present price takes
// the shorter one of each.  It is wrong where twice as many tiles of half the width are dearer than it has them (E 4, H 1088, F 8128,
// T = 412 133 / 143).
struct Shorten { int n_up = 0, n_down = 0, k_up = 0, k_down = 0; };   // full-width N tiles of the launches; n_up = 0: tiles as given
constexpr int SHORT_TILE_ROWS = 192;
constexpr int EPILOGUE_UP = 4 * 32, EPILOGUE_DOWN = 24 * 32;          // in units of K

// `tall`, `shortened`: M tiles of 256 and of SHORT_TILE_ROWS rows
constexpr int64_t launch_cost(int64_t tiles, int k) { return (half_width_pays(tiles) ? 10 : 16 * ((tiles + 255) >> 8)) * (int64_t)k; }
constexpr int64_t routed_cost(const Shorten& s, int64_t m_tiles) {
  return launch_cost(m_tiles * s.n_up, s.k_up + EPILOGUE_UP) + launch_cost(m_tiles * s.n_down, s.k_down + EPILOGUE_DOWN);
}
constexpr bool short_tiles_pay(const Shorten& s, int64_t tall, int64_t shortened) {
  return 13 * routed_cost(s, shortened) < 16 * routed_cost(s, tall);
}

// Slabs of K that the fp32 expert GEMM fetches ahead.  Two keep `of_two` workgroups of its tile on a compute unit, one lets
// `of_one` of them fit: one where that saves a round of `tiles` on 256 compute units.  us per call, two / one.  64 x 128 tiles (2, 3):
// skipping forward, nothing skipped, E 16, H 1024, F 512, T = 2000 (560 in either launch) 216 / 213, T = 2750 (752) 244 / 218; E 4, H 512,
// F 512, T = 3000 (766) 140 / 119, T = 3300 (840: two rounds both ways) 145 / 147, T = 4000 (1016) 145 / 157.  32 x 128 tiles (2, 4): the
// same, E 8, H 1024, F 256, up, T = 2000 (516) 107 / 105, T = 2700 (688) 139 / 129.  The routed counts are expected ones, and where either
// takes several rounds the rule can be wrong by a few per cent (E 8, H 512, F 1024, T = 2400 187 / 196).
constexpr int f32_slabs_ahead(int64_t tiles, int of_two, int of_one) {
  return (tiles + 256 * of_two - 1) / (256 * of_two) > (tiles + 256 * of_one - 1) / (256 * of_one) ? 1 : 2;
}
// Whether the column tiles of an fp32 launch are the fastest in the grid.  A routed launch has row tiles without rows, the last ones,
// and with the row tiles fastest they come once per column tile: the workgroups that have work are dealt to the compute units unevenly.
// us per call, row / column tiles fastest, threshold 0.6: E 4, H 864, F 768, top-4, T = 653 135 / 82; E 8, H 388, F 1792, top-6, T = 1657
// 248 / 190; nothing skipped: E 8, H 1024, F 256, T = 2000 126 / 105; E 4, H 180, F 324, T = 956 38 / 39.  Dense launches have no such
// tiles: 91 passes of all experts by columns took 1.00 of the time, the worst 1.08.
constexpr int64_t GRID_Y_MAX = 65535;
constexpr bool f32_columns_first(bool routed, int64_t row_tiles) { return routed && row_tiles <= GRID_Y_MAX; }
// Row tiles of a routed launch, expected: every expert's last one is half full.
constexpr int64_t routed_row_tiles(int64_t rows, int experts, int tile_rows) { return (rows + (int64_t)experts * (tile_rows / 2)) / tile_rows; }

}  // namespace moep
