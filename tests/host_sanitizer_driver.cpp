// Host logic of libmoeprune under AddressSanitizer / UndefinedBehaviorSanitizer: subset rank / unrank, workspace
// planning and the argument-error paths of every entry point.  No kernel is launched and no GPU is needed: every
// call below either is pure host arithmetic or must be refused before it reaches the HIP runtime.
// Built and run by tests/test_host_sanitizers.py against the sanitized build of the library.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "enum_plan.h"
#include "moeprune.h"
#include "skip_plan.h"
#include "tile_plan.h"

static int failures = 0;
#define EXPECT(cond)                                                          \
  do {                                                                        \
    if (!(cond)) { ++failures; std::printf("FAILED line %d: %s\n", __LINE__, #cond); } \
  } while (0)

static int64_t binom(int n, int r) {
  if (r < 0 || r > n) return 0;
  int64_t c = 1;
  for (int i = 1; i <= r; ++i) c = c * (n - r + i) / i;
  return c;
}

int main() {
  // ---- subsets: every index of every (E, r) up to E = 14, plus the corners of E = 32
  for (int E = 1; E <= 14; ++E)
    for (int r = 1; r <= E; ++r) {
      const int64_t n = moep_num_subsets(E, r);
      EXPECT(n == binom(E, r));
      uint32_t prev = 0;
      for (int64_t i = 0; i < n; ++i) {
        uint32_t m = 0;
        EXPECT(moep_subset_unrank(E, r, i, &m) == MOEP_OK);
        EXPECT(__builtin_popcount(m) == r && (E == 32 || (m >> E) == 0));
        EXPECT(moep_subset_rank(E, r, m) == i);
        if (i > 0) {   // lexicographic order of the sorted tuples = descending order of the bit-reversed masks
          uint32_t a = __builtin_bitreverse32(prev), b = __builtin_bitreverse32(m);
          EXPECT(a > b);
        }
        prev = m;
      }
    }
  {
    uint32_t m = 0;
    EXPECT(moep_num_subsets(32, 16) == binom(32, 16));
    EXPECT(moep_subset_unrank(32, 16, moep_num_subsets(32, 16) - 1, &m) == MOEP_OK && m == 0xffff0000u);
    EXPECT(moep_subset_rank(32, 16, 0xffff0000u) == moep_num_subsets(32, 16) - 1);
    EXPECT(moep_subset_unrank(32, 32, 0, &m) == MOEP_OK && m == 0xffffffffu);
    EXPECT(moep_subset_unrank(32, 1, 31, &m) == MOEP_OK && m == 0x80000000u);
    EXPECT(moep_subset_unrank(8, 2, 28, &m) == MOEP_EINVAL && std::strlen(moep_last_error()) > 0);
    EXPECT(moep_subset_unrank(8, 2, -1, &m) == MOEP_EINVAL);
    EXPECT(moep_subset_unrank(8, 2, 0, nullptr) == MOEP_EINVAL);
    EXPECT(moep_num_subsets(0, 1) == -1 && moep_num_subsets(33, 2) == -1 && moep_num_subsets(8, 9) == -1);
    EXPECT(moep_subset_rank(8, 2, 0x7) == -1 && moep_subset_rank(8, 2, 0x101) == -1);
  }

  // ---- workspace planning over a grid of shapes, including the largest and degenerate ones
  const int64_t Ts[] = {0, 1, 255, 256, 257, 16384, 262144, (int64_t)1 << 30, -1, ((int64_t)1 << 30) + 1};
  const int Es[] = {0, 1, 2, 8, 16, 32, 33};
  for (int64_t T : Ts)
    for (int E : Es)
      for (moep_dtype dt : {MOEP_F32, MOEP_BF16}) {
        const size_t w1 = moe_expert_outputs_workspace(T, E, 4096, 14336, dt);
        const size_t w2 = moe_forward_skip_workspace(T, E, 4096, 14336, dt);
        const size_t w3 = moe_expert_outputs_packed_workspace(T, E, 4096, 14336, dt);
        const bool ok = T >= 0 && T <= ((int64_t)1 << 30) && E >= 1 && E <= 32;
        EXPECT(ok || (w1 == 0 && w2 == 0 && w3 == 0));
        for (int k : {1, 2, 4})
          for (int r = 0; r <= E + 1 && r <= 33; ++r) {
            const size_t we = prune_enumerate_workspace(T, E, 4096, k, r, dt);
            const bool ok_e = ok && k <= E && r >= 1 && r <= E && binom(E, r) <= ((int64_t)1 << 24);
            EXPECT(ok_e ? we >= 256 : we == 0);
          }
        for (int k : {0, 1, 4, 16, 17}) (void)moe_forward_skip_topk_workspace(T, E, 4096, 14336, dt, k);
        for (int n : {0, 1, 6, 16, 17}) (void)moe_expert_outputs_ranked_workspace(T, E, 4096, 14336, dt, n);
      }
  {
    const int rs[] = {6, 4, 8, 1};
    EXPECT(prune_enumerate_multi_workspace(262144, 8, 4096, 2, 4, rs, MOEP_BF16) >=
           prune_enumerate_workspace(262144, 8, 4096, 2, 4, MOEP_BF16));
    EXPECT(prune_enumerate_multi_workspace(262144, 8, 4096, 2, 0, rs, MOEP_BF16) == 0);
    EXPECT(prune_enumerate_multi_workspace(262144, 8, 4096, 2, 4, nullptr, MOEP_BF16) == 0);
    EXPECT(moe_packed_weights_bytes(8, 4096, 14336, MOEP_BF16) == (size_t)8 * 3 * 4096 * 14336 * 2);
    EXPECT(moe_packed_weights_bytes(8, 4096, 14336, MOEP_F32) == 0 && moe_packed_weights_bytes(8, 100, 64, MOEP_BF16) == 0);
    EXPECT(skip_calibrate_beta_workspace(0) == 0 && skip_calibrate_beta_workspace(1) > 0);
  }

  // ---- plans of the subset enumeration: the token tiles cover the batch, their partial sums lie within the workspace in front
  // of what follows them, and the table scorers add at most 1024 tokens in fp32 before the fp64 sum over the tiles (with more
  // than 16 experts as long as the tiles fit the grid's second dimension).  Every plan of the table scorers has a kernel.
  const int64_t plan_Ts[] = {1, 7, 33, 777, 4096, 5000, 16384, 65536, 262144, 524289, ((int64_t)1 << 20) + 1, (int64_t)5 << 20, (int64_t)1 << 26};
  for (int E = 1; E <= 32; ++E)
    for (int k = 1; k <= E && k <= 16; ++k)
      for (int r = 1; r <= E; ++r) {
        if (binom(E, r) > ((int64_t)1 << 24)) continue;
        for (int64_t T : plan_Ts) {
          moep::EnumPlan q;
          EXPECT(moep::plan_enumerate(T, E, 64, k, r, &q) == MOEP_OK);
          EXPECT(q.tok_tile >= 1 && q.n_tok_tiles * q.tok_tile >= T && (q.n_tok_tiles - 1) * q.tok_tile < T);
          const size_t sums = (size_t)q.n_tok_tiles * q.n_sub * sizeof(float);
          EXPECT(q.off_partial + sums <= (q.fused_threads ? q.off_sel : q.off_partial_cnt) && q.off_sel <= q.total);
          EXPECT((q.fused_threads != 0) == (q.use_lut && E <= 16));
          if (q.fused_threads) {
            EXPECT(q.fused_threads >= 256 && q.fused_threads <= 1024 && q.fused_lds <= 64 * 1024 && q.tok_tile % q.fused_tg == 0);
            EXPECT(q.n_act >= 4 && q.n_act <= 12 && (q.fused_spl == 4 || (q.fused_spl == 14 && q.n_act > 4)));
          } else if (q.use_lut) {
            EXPECT(q.n_act >= 4 && q.n_act <= 12);
          }
          if (q.use_lut) EXPECT(q.tok_tile <= 1024 || (!q.fused_threads && T > (int64_t)65535 * 1024));
        }
      }

  // ---- records written by the Gram pass: few tokens or long rows, and only where those of every r fit beside their sums
  {
    auto records = [](int64_t T, int E, int H, int k, std::vector<int> rs, moep_dtype dt = MOEP_BF16, int n_rank = 0) {
      std::vector<moep::EnumPlan> q(rs.size());
      std::vector<const moep::EnumPlan*> at;
      for (size_t i = 0; i < rs.size(); ++i) {
        EXPECT(moep::plan_enumerate(T, E, H, k, rs[i], &q[i]) == MOEP_OK);
        at.push_back(&q[i]);
      }
      const size_t room = prune_enumerate_multi_workspace(T, E, H, k, (int)rs.size(), rs.data(), dt);
      moep::RecordPlan r;
      if (!moep::records_by_gram_pass(at.data(), (int)rs.size(), n_rank, dt == MOEP_F32, room, &r)) return false;
      size_t end = 0;                                // nothing overlaps, everything lies in the workspace
      for (size_t i = 0; i < rs.size(); ++i) {
        const size_t sums = (size_t)q[i].n_tok_tiles * q[i].n_sub * 4;
        EXPECT(r.rec[i] >= end && r.rec[i] % 256 == 0);
        EXPECT(r.partial[i] >= r.rec[i] + (size_t)T * q[i].rec_floats * 4 && r.partial[i] % 256 == 0);
        EXPECT(r.cnt[i] >= r.partial[i] + sums && r.cnt[i] % 256 == 0);
        end = r.cnt[i] + (q[i].fused_threads ? 0 : sums);
        EXPECT(end <= room);
      }
      return true;
    };
    EXPECT(records(4608, 16, 64, 2, {14}) && !records(4609, 16, 64, 2, {14}));                   // a tile per token, 4 active ranks
    EXPECT(records(6912, 16, 64, 4, {12}) && !records(6913, 16, 64, 4, {12}));                   // 8
    EXPECT(records(9216, 16, 64, 8, {15}) && !records(9217, 16, 64, 8, {15}));                   // 9
    EXPECT(records(11520, 16, 64, 2, {14, 12}) && !records(11521, 16, 64, 2, {14, 12}));         // 4 and 6
    EXPECT(records(9216, 8, 64, 2, {7}) && !records(9217, 8, 64, 2, {7}));                       // two tokens to a tile
    EXPECT(records(18432, 4, 64, 2, {2}) && !records(18433, 4, 64, 2, {2}));                     // four
    EXPECT(records(65536, 16, 1024, 2, {14}) && !records(65536, 16, 960, 2, {14}));              // rows long enough
    EXPECT(records(65536, 8, 1024, 2, {6, 4}, MOEP_F32) && !records(65536, 8, 960, 2, {6, 4}, MOEP_F32));
    EXPECT(!records(32000, 9, 2048, 2, {6}, MOEP_F32) && records(32000, 9, 2048, 2, {6}));       // seven rows of padding
    EXPECT(records(15360, 16, 64, 4, {12}, MOEP_BF16, 8) && !records(15361, 16, 64, 4, {12}, MOEP_BF16, 8));   // 8 ranked rows per token
    EXPECT(records(12288, 4, 64, 2, {2}, MOEP_BF16, 4) && !records(12289, 4, 64, 2, {2}, MOEP_BF16, 4));       // 4
    EXPECT(records(10752, 16, 64, 4, {12}, MOEP_BF16, 9) && !records(10753, 16, 64, 4, {12}, MOEP_BF16, 9));   // 9
    EXPECT(!records(65536, 2, 4096, 1, {1}, MOEP_BF16, 2) && records(65536, 3, 704, 2, {2}, MOEP_BF16, 3));    // 2 and 3: padding
    EXPECT(records(40000, 16, 512, 4, {12}, MOEP_BF16, 8) && !records(40000, 16, 448, 4, {12}, MOEP_BF16, 8));
    EXPECT(records(700, 8, 192, 2, {5, 6, 7}) && records(700, 8, 192, 1, {5, 6, 7, 8}));         // three and four r that fit
    EXPECT(!records(5600, 8, 192, 2, {4, 6, 7, 1}) && !records(700, 8, 192, 2, {4, 6, 7, 1}));   // four that do not
    EXPECT(!records(700, 8, 192, 1, {5, 6, 7, 8, 7}) && !records(100, 17, 64, 2, {16}) && !records(0, 8, 64, 2, {6}));
  }

  // ---- tiles of a routed call: shorter ones where they make it shorter (us of whole calls, 256 / 192 rows, at tile_plan.h)
  {
    auto pays = [](int H, int F, int tall, int shortened) {
      return moep::short_tiles_pay({(F + 127) / 128, (H + 255) / 256, H, F}, tall, shortened);
    };
    EXPECT(pays(4096, 14336, 16, 16) && !pays(4096, 14336, 16, 20));         // two tiles per expert either way; half of them three
    EXPECT(pays(192, 4736, 16, 20) && pays(256, 1536, 23, 24));              // as many rounds
    EXPECT(pays(128, 8640, 33, 48) && pays(512, 9408, 16, 18));              // more, short of what the shorter steps save
    // a third round, or a second, of a few steps and a whole epilogue
    EXPECT(!pays(3136, 128, 32, 45) && !pays(1664, 64, 32, 54) && !pays(1984, 128, 32, 40) && !pays(1920, 64, 64, 79));
  }

  // ---- a last round of up to 128 tiles in half the width: from two rounds on, K deep enough, more than 128 rows, and a table that holds both
  {
    auto tail = [](int64_t tiles, int k = 1024, int row_groups = 8, int n_half = 16) { return moep::tail_tiles(tiles, 8, n_half, k, row_groups); };
    EXPECT(tail(1) == 0 && tail(128) == 0 && tail(256) == 0 && tail(257) == 1 && tail(384) == 128 && tail(385) == 0 && tail(511) == 0);
    EXPECT(tail(512) == 0 && tail(513) == 1 && tail(640) == 128 && tail(641) == 0);
    EXPECT(tail(300, 1023) == 0 && tail(300, 1024) == 44 && tail(300, 1024, 6) == 44 && tail(300, 1024, 4) == 0);
    EXPECT(tail(300, 1024, 8, 8) == 0 && tail(300, 1024, 8, 15) == 44);
    for (int n_full = 1; n_full <= 200; ++n_full)
      for (int n_half : {2 * n_full - 1, 2 * n_full})
        for (int64_t m_tiles = 1; m_tiles <= 600; ++m_tiles) {
          const int64_t tiles = m_tiles * n_full, t = moep::tail_tiles(tiles, n_full, n_half, 4096, 8);
          EXPECT(t >= 0 && t <= 128 && tiles + t <= m_tiles * n_half);
          if (t) EXPECT((tiles - t) % 256 == 0 && tiles - t >= 256);
        }
  }

  // ---- weights of a routed call that are loaded past the caches: of the kept experts, not of the layer (gate/up 738 MB, 184 MB of
  // four experts, 92 MB of two; down half of that)
  {
    auto streams = [](int kept, bool gate_up) {
      moep::SkipPlan q;
      EXPECT(moep::plan_skip(42 * kept, 16, 2048, 5632, MOEP_BF16, 2, kept, &q) == MOEP_OK && !q.few && q.kept_experts == kept);
      return moep::routed_weights_stream(q, gate_up);
    };
    EXPECT(streams(16, true) && streams(5, true) && !streams(4, true) && !streams(2, true));
    EXPECT(streams(16, false) && streams(9, false) && !streams(8, false) && !streams(2, false));
  }

  // ---- slabs ahead in the fp32 GEMM: one where a third (64-row tiles) or a third and fourth workgroup per compute unit saves a round
  {
    auto tall = [](int64_t tiles) { return moep::f32_slabs_ahead(tiles, 2, 3); };
    auto low = [](int64_t tiles) { return moep::f32_slabs_ahead(tiles, 2, 4); };
    EXPECT(tall(1) == 2 && tall(512) == 2 && tall(513) == 1 && tall(768) == 1 && tall(769) == 2 && tall(1024) == 2 && tall(1025) == 1);
    for (int64_t tiles : {1500, 1536, 1537, 2048, 4000, 100000}) EXPECT(tall(tiles) == 1);
    EXPECT(low(512) == 2 && low(513) == 1 && low(1024) == 1);
    EXPECT(moep::routed_row_tiles(4000, 4, 64) == 64 && moep::routed_row_tiles(4000, 8, 64) == 66 && moep::routed_row_tiles(3000, 8, 32) == 97);
    EXPECT(moep::f32_columns_first(true, 1) && moep::f32_columns_first(true, 65535) && !moep::f32_columns_first(true, 65536) && !moep::f32_columns_first(false, 8));
    EXPECT(moep::routed_row_tiles(1, 1, 64) == 0 && moep::routed_row_tiles((int64_t)1 << 31, 32, 32) == ((int64_t)1 << 26) + 16);
  }

  // ---- tokens dispatched by one workgroup: a thread each, 256 at least
  for (int E = 2; E <= 32; ++E)
    for (int k = 1; k <= 16; ++k) {
      const int most = moep::dispatch_one_tokens(E, k);
      EXPECT(most >= 256 && most <= moep::DISPATCH_ONE_MAX && (k == 1 || most <= moep::dispatch_one_tokens(E, k - 1)));
    }
  EXPECT(moep::dispatch_one_tokens(8, 2) == 1024 && moep::dispatch_one_tokens(16, 4) == 512 && moep::dispatch_one_tokens(32, 2) == 512);
  EXPECT(moep::dispatch_one_tokens(24, 6) == 256 && moep::dispatch_one_tokens(32, 16) == 256 && moep::dispatch_one_tokens(16, 16) == 256);

  // ---- argument errors: every call must come back with a status and a message, having launched nothing
  void* p = (void*)(uintptr_t)(1 << 20);          // never dereferenced on the host
  float* fp = (float*)p;
  int32_t* ip = (int32_t*)p;
  uint32_t* up = (uint32_t*)p;
  EXPECT(moe_expert_outputs(p, p, p, p, p, 16, 0, 64, 64, MOEP_BF16, fp, p, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_expert_outputs(p, p, p, p, p, 16, 4, 60, 64, MOEP_BF16, fp, p, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(moe_expert_outputs(p, nullptr, p, p, p, 16, 4, 64, 64, MOEP_BF16, fp, p, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_expert_outputs(p, p, p, p, p, 16, 4, 64, 64, MOEP_BF16, fp, p, nullptr, 0, nullptr) == MOEP_EWORKSPACE);
  EXPECT(moe_expert_outputs(p, p, p, p, p, 16, 4, 64, 64, MOEP_BF16, fp, p, (char*)p + 8, (size_t)1 << 30, nullptr) == MOEP_EWORKSPACE);
  EXPECT(moe_expert_outputs(p, p, p, p, p, 16, 4, 64, 64, MOEP_BF16, fp, p, p, 16, nullptr) == MOEP_EWORKSPACE);
  EXPECT(moe_expert_outputs(p, p, p, p, p, 0, 4, 64, 64, MOEP_BF16, fp, p, nullptr, 0, nullptr) == MOEP_OK);   // empty batch
  EXPECT(moe_expert_outputs_packed(p, p, nullptr, 16, 4, 64, 64, MOEP_BF16, fp, p, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_expert_outputs_packed(p, p, p, 16, 4, 64, 64, MOEP_F32, fp, p, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate(fp, p, 16, 8, 64, MOEP_BF16, 2, 9, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate(fp, p, 16, 8, 64, MOEP_BF16, 0, 4, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate(fp, p, 16, 32, 64, MOEP_BF16, 2, 16, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate(fp, p, 16, 8, 100, MOEP_BF16, 2, 4, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate(fp, p, 16, 8, 64, MOEP_BF16, 2, 4, nullptr, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate(nullptr, p, 16, 8, 64, MOEP_BF16, 2, 4, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate(fp, p, 16, 8, 64, MOEP_BF16, 2, 4, fp, ip, up, nullptr, p, 16, nullptr) == MOEP_EWORKSPACE);
  {
    const int rs[] = {6, 9};
    EXPECT(prune_enumerate_multi(fp, p, 16, 8, 64, MOEP_BF16, 2, 2, rs, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
    EXPECT(prune_enumerate_multi(fp, p, 16, 8, 64, MOEP_BF16, 2, 0, rs, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  }
  // Eq. 3 as written: its limits are argument errors, found before anything touches the GPU
  EXPECT(prune_enumerate_direct_workspace(262144, 8, 4096, 2, 4, MOEP_BF16) >= 512u * 70 * 8);
  EXPECT(prune_enumerate_direct_workspace(262144, 16, 2048, 4, 8, MOEP_BF16) == 0);            // 12870 subsets
  EXPECT(prune_enumerate_direct(fp, p, 16, 16, 64, MOEP_BF16, 4, 8, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate_direct(fp, p, 16, 16, 64, MOEP_BF16, 5, 15, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate_direct(fp, p, 16, 8, 16384, MOEP_BF16, 2, 6, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate_direct(fp, p, 16, 8, 70, MOEP_F32, 2, 6, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(prune_enumerate_direct(fp, p, 16, 8, 64, MOEP_BF16, 2, 9, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate_direct(fp, p, 16, 8, 64, MOEP_BF16, 2, 6, nullptr, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate_direct(fp, nullptr, 16, 8, 64, MOEP_BF16, 2, 6, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate_direct(fp, p, 16, 8, 64, MOEP_BF16, 2, 6, fp, ip, up, nullptr, p, 16, nullptr) == MOEP_EWORKSPACE);
  EXPECT(prune_enumerate_static(fp, p, 200000, 8, 64, MOEP_BF16, 2, 4, fp, ip, up, nullptr, nullptr) == MOEP_EWORKSPACE);
  EXPECT(prune_enumerate_static(fp, p, 100, 8, 64, MOEP_BF16, 2, 4, nullptr, ip, up, nullptr, nullptr) == MOEP_EINVAL);
  EXPECT(prune_enumerate_ranked(fp, ip, ip, p, 16, 8, 64, MOEP_BF16, 4, 2, 4, fp, ip, up, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  uint8_t* bp = (uint8_t*)p;
  EXPECT(moe_forward_skip(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 3, 0.5f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(moe_forward_skip(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 2, -1.0f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_forward_skip(p, p, p, p, p, 16, 1, 64, 64, MOEP_BF16, 2, 0.5f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_forward_pruned_skip(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 2, 0x100u, 0.5f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_forward_pruned_skip(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 2, 0x1u, 0.5f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_forward_pruned_skip_packed(p, p, nullptr, 16, 8, 64, 64, MOEP_BF16, 2, 0xffu, 0.5f, p, bp, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_forward_skip_topk(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 17, 0xffu, 0.1f, p, ip, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(moe_forward_skip_topk(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 4, 0x7u, 0.1f, p, ip, nullptr, nullptr, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moe_pack_weights(p, p, p, 8, 64, 64, MOEP_F32, p, nullptr) == MOEP_EUNSUPPORTED);
  EXPECT(moe_pack_weights(p, p, p, 8, 64, 64, MOEP_BF16, (char*)p + 16, nullptr) == MOEP_EINVAL);
  EXPECT(skip_calibrate_beta(fp, 0, 8, 0xffu, fp, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(skip_calibrate_beta(fp, 16, 8, 0x1u, fp, p, 1 << 20, nullptr) == MOEP_EINVAL);
  int64_t* lp = (int64_t*)p;
  EXPECT(expert_selection_stats(fp, 16, 8, 9, 4, lp, lp, up, nullptr) == MOEP_EINVAL);
  EXPECT(expert_selection_stats(fp, 16, 8, 2, 0, lp, lp, up, nullptr) == MOEP_EINVAL);
  EXPECT(moe_expert_outputs_ranked(p, p, p, p, p, 16, 8, 64, 64, MOEP_BF16, 9, fp, ip, ip, p, p, 1 << 20, nullptr) == MOEP_EINVAL);
  EXPECT(moep_mfma_ceiling(p, p, 1 << 20, 3, fp, 1 << 20, nullptr, nullptr) == MOEP_EINVAL);
  {
    const char* names[4]; double ms[4]; int64_t cnt[4]; float f[4];
    EXPECT(moep_timing_collect(nullptr, ms, cnt, 4) == -1);
    EXPECT(moep_timing_collect(names, ms, cnt, 4) == 0);       // nothing recorded
    EXPECT(moep_timing_records(names, f, 0) == -1);
    EXPECT(moep_timing_records(names, f, 4) == 0);
  }
  EXPECT(std::strlen(moep_last_error()) > 0);
  std::printf(failures ? "host sanitizer driver: %d check(s) failed\n" : "host sanitizer driver: all checks passed\n", failures);
  return failures ? 1 : 0;
}
