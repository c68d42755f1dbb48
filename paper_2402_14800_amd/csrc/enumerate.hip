// Enumeration of kept-expert subsets (Sec. 3.2, Eq. 3) through the per-token Gram matrix.
//
// For token t let Y_t be the E x H matrix of its expert outputs, a the Eq. 1 weights of the full
// layer (top-k of all experts) and b those of the layer pruned to the kept set C (top-min(k,r)
// of C).  Then F'(x_t,C) - F(x_t) = sum_e (b_e - a_e) Y_t[e,:] and its squared norm is d^T G_t d
// with d = b - a, G_t = Y_t Y_t^T.  The kernels:
//
//   gram        G_t for every token: the only pass over Y (HBM-bound).  bf16: rows are fetched in whole
//               1 KB pieces, turned into MFMA fragments through wave-private LDS, and multiplied with
//               one v_mfma_f32_16x16x32_bf16 per 16 rows x 32 hidden units, the SAME registers feeding
//               both operands (B = A^T); two tokens per tile when E <= 8.
//   prep        per token: stable descending order of the logits (ties -> lower index), and
//               everything the scorer needs, moved to RANK space (position j = j-th ranked expert):
//               exp(l_j - l_0), l_j, the full-layer weights a_j, the Gram matrix permuted to rank
//               order (off-diagonals doubled).  Only the first n_act = min(E, min(k,r) + E - r)
//               positions can ever be selected by a pruned layer, so only those are kept.
//   score       lane = subset, loop over a tile of tokens.  Per token all data is wave-uniform
//               (scalar loads); each lane walks the rank positions, takes the first min(k,r) whose
//               expert is in its mask, forms d explicitly and evaluates d^T G d.  A pair whose
//               selection equals the full top-k contributes exactly 0 and is counted.
//   score (many subsets; up to 16 experts through fused_score_lut_kernel, which keeps the tables in LDS)
//               A token's error depends on the subset only through WHICH of its first n_act ranked experts are kept, and
//               then only through the first min(k,r) of those: C(n_act, min(k,r)) possible selections per token against
//               C(E,r) subsets (495 against 12870 for E = 16, k = 4, r = 8).  qtable evaluates the error of every selection once per token; score_lut then needs, per (subset, token), a few table look-ups:
//               kept mask -> pattern of kept rank positions (nibble tables built per token from its order),
//               pattern -> selection index (one table per launch), selection index -> error.
//   reduce      loss[i] = sum over token tiles of the partial sums, in a fixed order (fp64 adds).
//   argmin      lowest index attaining the minimum; its mask by lexicographic unranking.
#include "common.h"

namespace moep {
namespace {

// ------------------------------------------------------------------ binomials / unranking
struct BinomTable {
  uint32_t v[33][33];
  constexpr BinomTable() : v{} {
    for (int n = 0; n <= 32; ++n) {
      v[n][0] = 1;
      for (int r = 1; r <= n; ++r) v[n][r] = v[n - 1][r - 1] + (r <= n - 1 ? v[n - 1][r] : 0);
    }
  }
};
__constant__ BinomTable c_binom = BinomTable();

// Kept mask of subset `idx` in lexicographic order of sorted r-tuples over {0..E-1}.
__device__ uint32_t unrank_device(int E, int r, uint32_t idx) {
  uint32_t mask = 0;
  int rem = r;
  for (int e = 0; e < E; ++e) {
    if (rem == 0) break;
    const uint32_t with_e = c_binom.v[E - 1 - e][rem - 1];
    if (idx < with_e) { mask |= 1u << e; --rem; }
    else idx -= with_e;
  }
  return mask;
}

__global__ __launch_bounds__(256) void masks_kernel(int E, int r, uint32_t n_sub, uint32_t* __restrict__ masks) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < n_sub) masks[i] = unrank_device(E, r, i);
}

// ------------------------------------------------------------------ record layout
// Per token, CAP = capacity >= n_act, all fp32 unless noted:
//   [0, CAP)            ex_j  = exp(l_j - l_0), l in rank order (0 beyond n_act)
//   [CAP, 2 CAP)        l_j
//   [2 CAP, 3 CAP)      a_j   = full-layer Eq. 1 weight of rank j (0 for j >= k)
//   [3 CAP, 3 CAP + CAP (CAP + 1) / 2)   Gram in rank order, row-major upper triangle,
//                       diagonal as is, off-diagonal entries doubled
//   then ceil(CAP / 4) words: expert index of rank j in byte j
__host__ __device__ constexpr int rec_tri(int cap) { return cap * (cap + 1) / 2; }
__host__ __device__ constexpr int rec_order_off(int cap) { return 3 * cap + rec_tri(cap); }
__host__ __device__ constexpr int rec_size(int cap) {
  return (rec_order_off(cap) + (cap + 3) / 4 + 3) & ~3;
}

// ------------------------------------------------------------------ Gram, bf16 (MFMA)
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// EPAD = rows reserved per token inside a 16-row MFMA tile (4, 8 or 16): 16 / EPAD tokens per tile, one
// tile per wavefront; the 8x8 (4x4) blocks of the 16x16 product that pair different tokens are discarded.
// RANKED: the rows are the outputs of each token's n best-ranked experts, addressed through
// slot_of[t, j], with experts[t, j] naming the expert; G keeps its expert indexing (see below).
//
// A wavefront fetches each of the tile's 16 rows in whole 1 KB pieces (64 lanes x 16 bytes of ONE row per
// load), so that a DRAM page is read in one go wherever the 16 rows lie: with E T H a power of two the
// expert rows of a token fall into the same DRAM bank, and fragment-shaped loads (64 bytes of each of
// 16 rows per instruction) keep re-opening 16 pages of that bank (measured 4.8 against 5.7 TB/s at E = 16).
// The pieces become MFMA fragments through a wave-private 16 KB of LDS (chunk c of row j at position
// c ^ j: the row-wise writes and the column-wise fragment reads are both free of bank conflicts); the next
// 16 loads are in flight in registers while the current block of 512 hidden units is multiplied.  The
// same registers serve as both MFMA operands (B = A^T).
// STREAM: Y is far larger than the caches, so its loads carry the non-temporal hint (measured 6.2 -> 6.8 TB/s at
// 17 GB and 5.6 -> 6.0 TB/s at 4.3 GB; a Y of a few hundred MB that the down projection has just written is
// better read with ordinary loads: 6.5 against 5.0 TB/s at 0.27 GB).
// 16 bytes of Y with the non-temporal hint: a stream read once, not worth a place in the caches.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_streaming(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// F32: rows of floats, four v_mfma_f32_16x16x4_f32 per 16-byte chunk and 16 rows (the same register as both operands again;
// fp32 products and sums); E 8, H 512, 1501 tokens 47 -> 9 us against a wavefront per token with a shuffle tree per
// pair of experts, which re-read every row E times.
//
// Records: for up to RECORD_SETS values of r the wavefront goes on to write its tokens' records itself, from the 16 x 16 products
// in its LDS, and the Gram matrices never go to memory (!RECORDS: they do, for the prep kernel).  With long rows the pass waits
// for memory with 128 KB in flight on every compute unit, which covers the extra work; E 16, H 2048, 65536 tokens, two r: this
// kernel 702 -> 706 us and the 35 + 24 us of prep_kernel gone, E 8, H 4096 716 -> 729 and 11 + 8 gone.  Long batches of short rows
// have nothing to cover it (records_pay in enum_plan.h).
struct RecordArgs {
  const float* logits;
  int n, k;
  struct { float* rec; unsigned long long* clear; int cap, n_act, floats; } set[RECORD_SETS];   // clear: counter to be zeroed, or NULL
};
__device__ __forceinline__ void wavefront_sync() {         // LDS written by other lanes of the wavefront
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool F32, int EPAD, bool RANKED, bool STREAM, bool RECORDS>
__global__ __launch_bounds__(256) void gram_kernel(const uint4* __restrict__ Y,
                                                        const int32_t* __restrict__ slot_of,
                                                        const int32_t* __restrict__ experts,
                                                        float* __restrict__ G, int64_t T, int E, int n,
                                                        int H, RecordArgs recs) {
  constexpr int TPT = 16 / EPAD, LPT = 4 * EPAD;           // tokens per tile, lanes per token
  __shared__ uint4 stage[4][16 * 64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
  const int64_t t0 = tile * TPT;
  if (RECORDS && blockIdx.x == 0 && threadIdx.x < RECORD_SETS && (int)threadIdx.x < recs.n && recs.set[threadIdx.x].clear)
    *recs.set[threadIdx.x].clear = 0ull;
  if (!RECORDS && t0 >= T) return;
  // Records: what they need beside the products is made while the first rows are on their way: per token (lane lt of token tq),
  // by rank, exp, logit, full-layer weight and row of the products, per 4 ranks the experts, and a word that stays 0; per set the
  // place of each word's value in those (or its row and column of the triangle).
  __shared__ uint32_t s_token[4][TPT][4 * 16 + 4 + 4];
  __shared__ uint16_t s_word[RECORD_SETS][rec_size(EPAD)];
  constexpr int AT_L = 16, AT_A = 32, AT_ROW = 48, AT_ORDER = 64, AT_ZERO = 68, TRIANGLE = 0x8000;
  const int tq = lane / LPT, lt = lane % LPT;
  const bool some = RECORDS && t0 + tq < T;
  const float logit = some && lt < E ? recs.logits[(t0 + tq) * E + lt] : 0.f;
  const int expert = RANKED && some && lt < n ? experts[(t0 + tq) * n + lt] : 0;
  uint4* st = stage[wave];
  const int chunks = H / (F32 ? 4 : 8);                 // 16-byte chunks per row
  const int nkb = (chunks + 63) / 64;                   // blocks of 1 KB of every row
  // row j of the tile: expert (rank position) j % EPAD of token t0 + j / EPAD; rows without data read as zeros
  const uint4* rowp[16];
  bool rvalid[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int e = j % EPAD;
    const int64_t t = t0 + j / EPAD;
    rvalid[j] = e < (RANKED ? n : E) && t < T;
    int64_t r = 0;
    if (rvalid[j]) r = RANKED ? (int64_t)slot_of[t * n + e] : (int64_t)e * T + t;
    rowp[j] = Y + r * chunks + lane;
  }
  const int row = lane & 15, kg = lane >> 4;
  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
  uint4 v[16];
#define MOEP_GRAM_FETCH(kb)                                                                     \
  _Pragma("unroll") for (int j = 0; j < 16; ++j)                                                \
    v[j] = !(rvalid[j] && (kb) * 64 + lane < chunks) ? make_uint4(0, 0, 0, 0)                    \
           : STREAM ? load_streaming(&rowp[j][(kb) * 64]) : rowp[j][(kb) * 64];
  MOEP_GRAM_FETCH(0)
  if constexpr (RECORDS) {
    uint32_t* const tok = s_token[wave][tq];
    float* const lg = (float*)st + tq * 64;                // (the stage is not in use yet)
    int* const rank_of = (int*)lg + 16;
    int* const place = (int*)lg + 32;                      // RANKED: expert -> its row
    if (lt < 16) {
      lg[lt] = logit;
      if (RANKED) place[lt] = 0;
    }
    wavefront_sync();
    if (RANKED && lt < n) place[expert] = lt;
    if (lt < 16) {                                         // rank = experts that precede this one (as in prep_kernel)
      int rank = 0;
#pragma unroll
      for (int f = 0; f < (RANKED ? 16 : EPAD); ++f) {
        const float lf = lg[f];
        rank += f < E && f != lt && (lf > logit || (lf == logit && f < lt)) ? 1 : 0;
      }
      rank_of[lt] = lt < E ? rank : 255;
    }
    wavefront_sync();
    if (lt < 16) {                                         // lane = rank
      int here = 0;
      float l = 0.f;
#pragma unroll
      for (int e = 0; e < (RANKED ? 16 : EPAD); ++e)
        if (rank_of[e] == lt) { here = e; l = lg[e]; }
      tok[AT_L + lt] = __float_as_uint(l);
      tok[AT_ROW + lt] = (uint32_t)(tq * EPAD + (RANKED ? place[here] : here));
      rank_of[lt] = here;
    }
    wavefront_sync();
    if (lt < 16) tok[lt] = __float_as_uint(expf(__uint_as_float(tok[AT_L + lt]) - __uint_as_float(tok[AT_L])));
    wavefront_sync();
    if (lt < 16) {
      float den = 0.f;
      for (int j = 0; j < recs.k; ++j) den += __uint_as_float(tok[j]);
      tok[AT_A + lt] = lt < recs.k ? __float_as_uint(__uint_as_float(tok[lt]) / den) : 0u;
      if (lt < 4) {
        uint32_t packed = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) packed |= (uint32_t)rank_of[4 * lt + b] << (8 * b);
        tok[AT_ORDER + lt] = packed;
        tok[AT_ZERO + lt] = 0u;
      }
    }
    for (int i = 0; i < recs.n; ++i) {
      const int cap = recs.set[i].cap, n_act = recs.set[i].n_act, w = threadIdx.x;
      const int order_at = rec_order_off(cap);
      uint32_t word = AT_ZERO;
      if (w < 3 * cap) {
        const int which = w < cap ? 0 : w < 2 * cap ? 1 : 2, j = w - which * cap;
        if (j < n_act) word = (uint32_t)(16 * which + j);
      } else if (w < order_at) {
        int j = w - 3 * cap, a = 0;                        // row a of the triangle, column a + j
        while (j >= cap - a) { j -= cap - a; ++a; }
        if (a + j < n_act) word = TRIANGLE | (uint32_t)(a | (a + j) << 4);
      } else if (w < order_at + (cap + 3) / 4) {
        const int q = w - order_at, left = n_act - 4 * q;  // experts of this word: all four, or the first ones
        if (left > 0) word = (uint32_t)(AT_ORDER + q) | (uint32_t)(left < 4 ? left : 0) << 8;
      }
      if (w < recs.set[i].floats) s_word[i][w] = (uint16_t)word;
    }
    __syncthreads();
    if (t0 >= T) return;
  }
  for (int kb = 0; kb < nkb; ++kb) {
#pragma unroll
    for (int j = 0; j < 16; ++j) st[j * 64 + (lane ^ j)] = v[j];
    if (kb + 1 < nkb) { MOEP_GRAM_FETCH(kb + 1) }
    // MFMA 16x16x32: lane l supplies row (l & 15) and 8 consecutive hidden units; which 8 is free as long as
    // every row agrees, here chunk 4 s + (l >> 4) of the block
#pragma unroll
    for (int s = 0; s < 16; s += 2) {
      const uint4 c0 = st[row * 64 + ((4 * s + kg) ^ row)], c1 = st[row * 64 + ((4 * (s + 1) + kg) ^ row)];
      if constexpr (F32) {
        const f32x4 a0 = __builtin_bit_cast(f32x4, c0), a1 = __builtin_bit_cast(f32x4, c1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[i], a0[i], acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[i], a1[i], acc1, 0, 0, 0);
        }
      } else {
        const bf16x8 a0 = __builtin_bit_cast(bf16x8, c0), a1 = __builtin_bit_cast(bf16x8, c1);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, a0, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, a1, acc1, 0, 0, 0);
      }
    }
  }
#undef MOEP_GRAM_FETCH
  // Accumulator layout of the 16x16 tile: register v of lane l = row 4 (l / 16) + v, column l % 16.
  const int col = lane & 15;
  if constexpr (RECORDS) {
    float* const g = (float*)st;                           // the products, in the place of the stage
    wavefront_sync();
#pragma unroll
    for (int vv = 0; vv < 4; ++vv) g[(4 * (lane >> 4) + vv) * 16 + col] = acc0[vv] + acc1[vv];
    wavefront_sync();
    if (t0 + tq >= T) return;
    const uint32_t* const tok = s_token[wave][tq];
    for (int i = 0; i < recs.n; ++i) {
      const int floats = recs.set[i].floats;
      uint32_t* const out = (uint32_t*)recs.set[i].rec + (t0 + tq) * floats;
      for (int w = lt; w < floats; w += LPT) {
        const uint32_t word = s_word[i][w];
        uint32_t v;
        if (word & TRIANGLE) {
          const uint32_t a = word & 15u, b = (word >> 4) & 15u;
          const float x = g[tok[AT_ROW + a] * 16 + tok[AT_ROW + b]];
          v = __float_as_uint(a == b ? x : 2.0f * x);
        } else {
          v = tok[word & 0xffu];
          if (word >> 8) v &= 0xffffffffu >> (8 * (4 - (word >> 8)));
        }
        out[w] = v;
      }
    }
    return;
  }
  const int cj = col % EPAD;
  const int64_t ct = t0 + col / EPAD;
  if (ct >= T || cj >= (RANKED ? n : E)) return;
  const int ce = RANKED ? experts[ct * n + cj] : cj;
#pragma unroll
  for (int vv = 0; vv < 4; ++vv) {
    const int r = 4 * (lane >> 4) + vv;
    const int rj = r % EPAD;
    if (r / EPAD == col / EPAD && rj < (RANKED ? n : E)) {
      const int re = RANKED ? experts[ct * n + rj] : rj;
      G[(ct * E + re) * E + ce] = acc0[vv] + acc1[vv];
    }
  }
}

// E in 17..32: one token per 32x32 tile.
__global__ __launch_bounds__(256) void gram_bf16_32_kernel(const uint4* __restrict__ Y,
                                                           float* __restrict__ G, int64_t T, int E,
                                                           int H) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int row = lane & 31, kg = lane >> 5;
  const bool valid = row < E;
  const int chunks = H / 8;
  const uint4* src = Y + ((int64_t)(valid ? row : 0) * T + t) * chunks + kg;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int steps = H / 16;
  for (int s0 = 0; s0 < steps; s0 += 4) {
    uint4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = valid ? src[(s0 + i) * 2] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, v[i]);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, a, acc, 0, 0, 0);
    }
  }
  const int col = lane & 31;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (r < E && col < E) G[(t * E + r) * E + col] = acc[v];
  }
}

// fp32, E in 17..32: one token per 32x32 tile, rows fetched and staged as above (32 KB of LDS per wavefront, two of them
// per workgroup): E 32, H 512, 300 tokens 580 -> 16 us against a shuffle tree per pair of experts.  (The same staging in
// bf16 was slower than the kernel above: E 20, H 1024, 2000 tokens 21 against 17 us.)
__global__ __launch_bounds__(128) void gram_f32_32_kernel(const uint4* __restrict__ Y, float* __restrict__ G, int64_t T, int E,
                                                      int H) {
  __shared__ uint4 stage[2][32 * 64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * 2 + wave;
  if (t >= T) return;
  uint4* st = stage[wave];
  const int chunks = H / 4;
  const int nkb = (chunks + 63) / 64;
  const uint4* const src = Y + t * chunks + lane;         // row e: e T rows further
  const int64_t row_step = T * chunks;
  const int row = lane & 31, kg = lane >> 5;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  uint4 v[32];
#define MOEP_GRAM_FETCH(kb)                                                                                  \
  _Pragma("unroll") for (int j = 0; j < 32; ++j)                                                             \
    v[j] = j < E && (kb) * 64 + lane < chunks ? src[j * row_step + (kb) * 64] : make_uint4(0, 0, 0, 0);
  MOEP_GRAM_FETCH(0)
  for (int kb = 0; kb < nkb; ++kb) {
#pragma unroll
    for (int j = 0; j < 32; ++j) st[j * 64 + (lane ^ j)] = v[j];
    if (kb + 1 < nkb) { MOEP_GRAM_FETCH(kb + 1) }
    // MFMA 32x32: lane l supplies row l % 32; chunk 2 s + (l / 32) of the block
#pragma unroll 8
    for (int s = 0; s < 32; ++s) {
      const f32x4 a = __builtin_bit_cast(f32x4, st[row * 64 + ((2 * s + kg) ^ row)]);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], a[i], acc, 0, 0, 0);
    }
  }
#undef MOEP_GRAM_FETCH
  const int col = lane & 31;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int r = 8 * (w >> 2) + 4 * (lane >> 5) + (w & 3);
    if (r < E && col < E) G[(t * E + r) * E + col] = acc[w];
  }
}

// ------------------------------------------------------------------ Gram, fp32 storage, rows of any length and alignment
__global__ __launch_bounds__(256) void gram_f32_kernel(const float* __restrict__ Y,
                                                       float* __restrict__ G, int64_t T, int E,
                                                       int H) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  for (int e = 0; e < E; ++e)
    for (int f = e; f < E; ++f) {
      const float* ye = Y + ((int64_t)e * T + t) * H;
      const float* yf = Y + ((int64_t)f * T + t) * H;
      float s = 0.f;
      for (int h = lane; h < H; h += 64) s = fmaf(ye[h], yf[h], s);
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0) {
        G[(t * E + e) * E + f] = s;
        G[(t * E + f) * E + e] = s;
      }
    }
}


// ------------------------------------------------------------------ Gram from ranked expert outputs
// The rank-limited expert pass stores, per token, only the outputs of its n best-ranked experts, as
// rows of Yr addressed through slot_of[t, j]; experts[t, j] names the expert.  G keeps its expert
// indexing: entry (e_i, e_j) of token t is written for the token's n ranked experts only, which is
// every entry the routing-prep kernel reads as long as n >= n_act.
__global__ __launch_bounds__(256) void gram_ranked_f32_kernel(const float* __restrict__ Yr,
                                                              const int32_t* __restrict__ slot_of,
                                                              const int32_t* __restrict__ experts,
                                                              float* __restrict__ G, int64_t T, int E,
                                                              int n, int H) {
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  for (int i = 0; i < n; ++i)
    for (int j = i; j < n; ++j) {
      const float* yi = Yr + (int64_t)slot_of[t * n + i] * H;
      const float* yj = Yr + (int64_t)slot_of[t * n + j] * H;
      float s = 0.f;
      for (int h = lane; h < H; h += 64) s = fmaf(yi[h], yj[h], s);
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0) {
        const int ei = experts[t * n + i], ej = experts[t * n + j];
        G[(t * E + ei) * E + ej] = s;
        G[(t * E + ej) * E + ei] = s;
      }
    }
}

// ------------------------------------------------------------------ records from Gram matrices
// One thread per token.  STAGED: the thread builds its record in LDS (rec_floats + 1 words apart: no bank conflicts)
// and the workgroup then writes its tokens' records, which are consecutive in memory, in 16-byte pieces; otherwise
// (records too large for the LDS) every thread writes its own record word by word.
// CAP = the record's capacity at compile time: the order then sits in registers and every Gram entry is fetched before the
// first is used (a run-time capacity made the gathers one long chain: 12 us per launch however few the tokens, now 8);
// 0 = run time, for the capacities whose unrolled form would not fit the registers.
// unaffected (may be NULL) is cleared for the counting that follows.
template <int EMAX, int CAP, bool STAGED>
__global__ __launch_bounds__(256) void prep_kernel(const float* __restrict__ logits,
                                                   const float* __restrict__ G,
                                                   float* __restrict__ rec, int64_t T, int E, bool vec,
                                                   int k, int n_act, int cap_rt, int rec_floats,
                                                   unsigned long long* __restrict__ unaffected) {
  extern __shared__ float stage[];
  const int cap = CAP ? CAP : cap_rt;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x;
  const int64_t t = t0 + threadIdx.x;
  if (unaffected && blockIdx.x == 0 && threadIdx.x == 0) *unaffected = 0ull;
  if (t < T) {
  float l[EMAX];
  load_logits<EMAX>(logits, t, E, vec, l);
  // rank of expert e = number of experts that precede it: larger logit, or equal and lower index
  int rank[EMAX];
#pragma unroll
  for (int e = 0; e < EMAX; ++e) {
    int c = 0;
#pragma unroll
    for (int f = 0; f < EMAX; ++f)
      if (f < E && f != e) c += (l[f] > l[e] || (l[f] == l[e] && f < e)) ? 1 : 0;
    rank[e] = e < E ? c : 255;
  }
  float* R = STAGED ? stage + threadIdx.x * (rec_floats + 1) : rec + t * rec_floats;
  uint32_t* Rord = (uint32_t*)(R + rec_order_off(cap));
  if constexpr (CAP > 0) {
    int ord[CAP];
    float lv[CAP], ex[CAP], g[rec_tri(CAP)];
#pragma unroll
    for (int j = 0; j < CAP; ++j) {
      ord[j] = 0;
      lv[j] = 0.f;
#pragma unroll
      for (int e = 0; e < EMAX; ++e)
        if (j < n_act && rank[e] == j) { ord[j] = e; lv[j] = l[e]; }
    }
    const float* Gt = G + t * E * E;
    int idx = 0;
#pragma unroll
    for (int i = 0; i < CAP; ++i)
#pragma unroll
      for (int j = i; j < CAP; ++j, ++idx) g[idx] = j < n_act ? Gt[ord[i] * E + ord[j]] : 0.f;
    float den = 0.f;
#pragma unroll
    for (int j = 0; j < CAP; ++j) {
      ex[j] = j < n_act ? expf(lv[j] - lv[0]) : 0.f;
      if (j < k) den += ex[j];               // (k <= n_act: every rank below k can be selected, or r < k and E = n_act)
    }
#pragma unroll
    for (int j = 0; j < CAP; ++j) {
      R[j] = ex[j];
      R[CAP + j] = lv[j];
      R[2 * CAP + j] = j < k ? ex[j] / den : 0.f;
    }
    idx = 0;
#pragma unroll
    for (int i = 0; i < CAP; ++i)
#pragma unroll
      for (int j = i; j < CAP; ++j, ++idx) R[3 * CAP + idx] = i == j ? g[idx] : 2.0f * g[idx];
#pragma unroll
    for (int w = 0; w < (CAP + 3) / 4; ++w) {
      uint32_t packed = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (4 * w + b < CAP) packed |= (uint32_t)ord[4 * w + b] << (8 * b);
      Rord[w] = packed;
    }
    for (int i = rec_order_off(CAP) + (CAP + 3) / 4; i < rec_size(CAP); ++i) R[i] = 0.f;
  } else {
  for (int i = 0; i < rec_floats; ++i) R[i] = 0.f;
  int ord[EMAX];
  float l0 = 0.f;
  for (int j = 0; j < n_act; ++j) {
    int oe = 0;
    float lv = 0.f;
#pragma unroll
    for (int e = 0; e < EMAX; ++e)
      if (rank[e] == j) { oe = e; lv = l[e]; }
    ord[j] = oe;
    if (j == 0) l0 = lv;
    R[j] = expf(lv - l0);
    R[cap + j] = lv;
  }
  float den = 0.f;
  for (int j = 0; j < k; ++j) den += R[j];
  for (int j = 0; j < k; ++j) R[2 * cap + j] = R[j] / den;
  int idx = 3 * cap;
  for (int i = 0; i < cap; ++i)
    for (int j = i; j < cap; ++j, ++idx)
      if (i < n_act && j < n_act) {
        const float g = G[(t * E + ord[i]) * E + ord[j]];
        R[idx] = i == j ? g : 2.0f * g;
      }
  for (int w = 0; w < (cap + 3) / 4; ++w) {
    uint32_t packed = 0;
    for (int b = 0; b < 4; ++b) {
      const int j = 4 * w + b;
      if (j < n_act) packed |= (uint32_t)ord[j] << (8 * b);
    }
    Rord[w] = packed;
  }
  }
  }
  if (STAGED) {
    __syncthreads();
    const int64_t left = T - t0;
    const int words = (int)(left < (int64_t)blockDim.x ? left : (int64_t)blockDim.x) * rec_floats;   // a multiple of 4
    float4* dst = (float4*)(rec + t0 * rec_floats);
    for (int q = 4 * threadIdx.x; q < words; q += 4 * blockDim.x) {
      const float* src = stage + (q / rec_floats) * (rec_floats + 1) + q % rec_floats;   // the 4 words are one token's
      dst[q >> 2] = make_float4(src[0], src[1], src[2], src[3]);
    }
  }
}

// ------------------------------------------------------------------ scoring
// EXACT: every one of the CAP rank positions is in use (n_act == CAP), which removes the
// per-position guards from the token loop.
// A token costs a lane a wait for its record (scalar loads) and a short dependent chain, so a tile is dealt to SCORE_STRANDS
// strands of wavefronts (threadIdx.y), whose sums are added in LDS in strand order (28 and 70 subsets, E 8: 2048
// tokens 46 -> 18 us for both, 262144 tokens 232 -> 131 us).  !STRANDS: one strand, nothing to hand over, the workgroups no
// larger than they have to be (1820 subsets of 16 ranks, 20000 tokens: 391 us through the other form, 357 so).
constexpr int SCORE_STRANDS = 8;
template <int CAP, bool EXACT, bool STRANDS>
__global__ __launch_bounds__(STRANDS ? 1024 : 256) void score_kernel(const float* __restrict__ rec, int64_t T,
                                                    int tok_tile, int E, int r, int kk, int kfull,
                                                    int n_act_rt, uint32_t n_sub,
                                                    float* __restrict__ partial,
                                                    uint32_t* __restrict__ partial_cnt) {
  constexpr int RS = rec_size(CAP);
  const int n_act = EXACT ? CAP : n_act_rt;
  constexpr int OFF_L = CAP, OFF_A = 2 * CAP, OFF_G = 3 * CAP, OFF_O = rec_order_off(CAP);
  const uint32_t sub = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = sub < n_sub;
  // Idle lanes keep every expert: their selection always equals the full one and costs nothing.
  const uint32_t mask = live ? unrank_device(E, r, sub) : 0xffffffffu;
  const uint32_t full_bits = kk != kfull ? 0u : (kfull >= 32 ? 0xffffffffu : (1u << kfull) - 1u);   // r < k: never "same"
  const int64_t t_begin = (int64_t)blockIdx.y * tok_tile;
  const int64_t t_end = t_begin + tok_tile < T ? t_begin + tok_tile : T;

  const int strand = STRANDS ? __builtin_amdgcn_readfirstlane((int)threadIdx.y) : 0, strands = STRANDS ? (int)blockDim.y : 1;

  float total = 0.f;
  uint32_t same_cnt = 0;
  for (int64_t t = t_begin + strand; t < t_end; t += strands) {
    const float* R = rec + t * RS;                       // wave-uniform
    const uint32_t* Rord = (const uint32_t*)(R + OFF_O);
    // Everything the selection needs is fetched up front, unconditionally (wave-uniform scalar
    // loads), so that no load sits behind a lane-dependent condition.
    float ex[CAP], aw[CAP];
    uint32_t ordw[(CAP + 3) / 4];
#pragma unroll
    for (int j = 0; j < CAP; ++j) { ex[j] = R[j]; aw[j] = R[OFF_A + j]; }
#pragma unroll
    for (int j = 0; j < (CAP + 3) / 4; ++j) ordw[j] = Rord[j];
    float w[CAP];
    float sum = 0.f;
    uint32_t bits = 0;
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < CAP; ++j) {
      w[j] = 0.f;
      if (j < n_act) {
        const uint32_t e = (ordw[j >> 2] >> (8 * (j & 3))) & 0xffu;
        const bool take = ((mask >> e) & 1u) && cnt < kk;
        cnt += take ? 1 : 0;
        bits |= take ? (1u << j) : 0u;
        w[j] = take ? ex[j] : 0.f;
        sum += w[j];
      }
    }
    if (sum < 1e-30f) {
      // Every selected logit lies far below the token's maximum: redo Eq. 1 relative to the
      // largest SELECTED logit (the first one taken), as the definition has it.
      float m = 0.f;
      bool have = false;
#pragma unroll
      for (int j = 0; j < CAP; ++j)
        if (j < n_act && ((bits >> j) & 1u) && !have) { m = R[OFF_L + j]; have = true; }
      sum = 0.f;
#pragma unroll
      for (int j = 0; j < CAP; ++j) {
        w[j] = (j < n_act && ((bits >> j) & 1u)) ? __expf(R[OFF_L + j] - m) : 0.f;
        sum += w[j];
      }
    }
    const float inv = __builtin_amdgcn_rcpf(sum);
    float d[CAP];
#pragma unroll
    for (int j = 0; j < CAP; ++j) d[j] = fmaf(w[j], inv, -aw[j]);
    float q = 0.f;
    int gi = OFF_G;
#pragma unroll
    for (int i = 0; i < CAP; ++i) {
      float u = 0.f;
#pragma unroll
      for (int j = i; j < CAP; ++j, ++gi) u = fmaf(R[gi], d[j], u);
      q = fmaf(d[i], u, q);
    }
    const bool same = bits == full_bits;
    same_cnt += (same && live) ? 1u : 0u;
    total += same ? 0.f : q;
  }
  if constexpr (STRANDS) {
    __shared__ float s_total[1024];
    __shared__ uint32_t s_same[1024];
    const int at = threadIdx.y * blockDim.x + threadIdx.x;
    s_total[at] = total;
    s_same[at] = same_cnt;
    __syncthreads();
    if (strand == 0)
      for (int w = 1; w < strands; ++w) {
        total += s_total[w * blockDim.x + threadIdx.x];
        same_cnt += s_same[w * blockDim.x + threadIdx.x];
      }
  }
  if (strand == 0 && live) {
    partial[(int64_t)blockIdx.y * n_sub + sub] = total;
    partial_cnt[(int64_t)blockIdx.y * n_sub + sub] = same_cnt;
  }
}

// ------------------------------------------------------------------ scoring through per-token selection tables
// More than 16 experts: half masks have up to 65536 patterns, too many for the tables of the fused scorer further down.
// Rank of the selection made by the kept-position pattern `pat` (bit j = the token's j-th ranked expert is kept):
// the first kk set bits, as a kk-subset of the n_act positions, indexed in lexicographic order (index 0 = positions
// 0 .. kk-1 = the selection of the full layer when kk = k).  Patterns with fewer than kk bits belong to no subset.
// selbits[i] = the positions of selection i (the pattern with exactly kk bits that has index i).
__global__ __launch_bounds__(256) void selidx_kernel(int n_act, int kk, uint16_t* __restrict__ sel,
                                                     uint16_t* __restrict__ selbits) {
  const uint32_t pat = blockIdx.x * 256 + threadIdx.x;
  if (pat >= (1u << n_act)) return;
  uint32_t idx = 0;
  int rem = kk;
  for (int j = 0; j < n_act && rem > 0; ++j) {
    if ((pat >> j) & 1u) --rem;
    else idx += c_binom.v[n_act - 1 - j][rem - 1];     // all selections whose next position is j come first
  }
  sel[pat] = rem == 0 ? (uint16_t)idx : (uint16_t)1;     // too few bits: only idle lanes look these up (never index 0)
  if (rem == 0 && __popc(pat) == kk) selbits[idx] = (uint16_t)pat;
}

// One workgroup per token: the error d^T G d of every selection (kk of the first n_act rank positions), the same
// arithmetic as score_kernel's.  Selection 0 is the full layer's when kk = kfull: exactly 0.
template <int CAP, bool EXACT>
__global__ __launch_bounds__(256) void qtable_kernel(const float* __restrict__ rec, int kk, int kfull, int n_act_rt,
                                                     int n_combo, const uint16_t* __restrict__ selbits,
                                                     float* __restrict__ qtab, int nib,
                                                     uint16_t* __restrict__ nibtab) {
  constexpr int RS = rec_size(CAP);
  const int n_act = EXACT ? CAP : n_act_rt;
  constexpr int OFF_L = CAP, OFF_A = 2 * CAP, OFF_G = 3 * CAP;
  const int64_t t = blockIdx.x;
  const float* R = rec + t * RS;                        // wave-uniform
  float ex[CAP], aw[CAP];
#pragma unroll
  for (int j = 0; j < CAP; ++j) { ex[j] = R[j]; aw[j] = R[OFF_A + j]; }
  for (int c = threadIdx.x; c < n_combo; c += blockDim.x) {
    const uint32_t bits = selbits[c];
    float w[CAP];
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < CAP; ++j) {
      w[j] = (j < n_act && ((bits >> j) & 1u)) ? ex[j] : 0.f;
      sum += w[j];
    }
    if (sum < 1e-30f) {                                  // see score_kernel
      float m = 0.f;
      bool have = false;
#pragma unroll
      for (int j = 0; j < CAP; ++j)
        if (j < n_act && ((bits >> j) & 1u) && !have) { m = R[OFF_L + j]; have = true; }
      sum = 0.f;
#pragma unroll
      for (int j = 0; j < CAP; ++j) {
        w[j] = (j < n_act && ((bits >> j) & 1u)) ? __expf(R[OFF_L + j] - m) : 0.f;
        sum += w[j];
      }
    }
    const float inv = __builtin_amdgcn_rcpf(sum);
    float d[CAP];
#pragma unroll
    for (int j = 0; j < CAP; ++j) d[j] = fmaf(w[j], inv, -aw[j]);
    float q = 0.f;
    int gi = OFF_G;
#pragma unroll
    for (int i = 0; i < CAP; ++i) {
      float u = 0.f;
#pragma unroll
      for (int j = i; j < CAP; ++j, ++gi) u = fmaf(R[gi], d[j], u);
      q = fmaf(d[i], u, q);
    }
    qtab[t * n_combo + c] = (c == 0 && kk == kfull) ? 0.f : q;
  }
  // The token's nibble tables, which turn a kept mask into a kept-position pattern four experts at a time: entry v
  // of nibble nb = the rank positions (below n_act) of the experts 4 nb + b with bit b of v set.  Stored as the low
  // or high half of a 32-bit word shared with the neighbouring token, so that one look-up serves two tokens.
  const uint32_t* ordw = (const uint32_t*)(R + rec_order_off(CAP));
  for (int q = threadIdx.x; q < nib * 16; q += blockDim.x) {
    const int nb = q >> 4, v = q & 15;
    uint32_t pat = 0;
    for (int j = 0; j < n_act; ++j) {
      const uint32_t e = (ordw[j >> 2] >> (8 * (j & 3))) & 0xffu;
      if ((int)(e >> 2) == nb && ((v >> (e & 3)) & 1)) pat |= 1u << j;
    }
    nibtab[((t >> 1) * (nib * 16) + q) * 2 + (t & 1)] = (uint16_t)pat;   // tokens 2 i and 2 i + 1 share a word
  }
}

// Lane = LUT_SPL subsets (their look-up addresses, one per subset and mask nibble, stay in registers), loop over a tile of
// tokens, LUT_TG tokens per barrier (double-buffered in LDS).  Per pair: one look-up per nibble of the kept mask (lanes of a
// wavefront hold neighbouring subsets: few distinct entries, no bank conflicts), one of the pattern's selection index, one of
// that selection's error.
constexpr int LUT_TG = 8, LUT_SPL = 8, LUT_MAX_ACT = 12, LUT_MAX_COMBO = 512;
// Where the pattern table keeps pattern `pat` in LDS: pattern bits 6..10 folded onto the bits that choose the bank.
// The patterns of a wavefront's 64 subsets differ in the few rank positions of the experts that vary among them, any
// of the n_act; left to bits 1..5 alone the bank would ignore the rest and they would queue on a few banks.
__device__ __forceinline__ uint32_t lut_swizzle(uint32_t pat) { return pat ^ ((pat >> 5) & 0x3eu); }

template <int NIB>             // nibbles of the kept mask: ceil(E / 4), 5 to 8
__global__ __launch_bounds__(256, 3) void score_lut_kernel(const float* __restrict__ qtab,
                                                        const uint32_t* __restrict__ nibtab,
                                                        const uint16_t* __restrict__ sel, int64_t T, int tok_tile,
                                                        int E, int r, int n_act, int n_combo, bool count_same,
                                                        uint32_t n_sub, float* __restrict__ partial,
                                                        uint32_t* __restrict__ partial_cnt) {
  constexpr int SPL = LUT_SPL, NT = NIB * 16;            // nibble-table entries per token
  __shared__ uint16_t s_sel[1 << LUT_MAX_ACT];
  __shared__ uint32_t s_nib[2][LUT_TG / 2 * NT];
  __shared__ float s_q[2][LUT_TG * LUT_MAX_COMBO];
  const int tid = threadIdx.x;
  for (int i = tid; i < (1 << n_act); i += 256) s_sel[lut_swizzle((uint32_t)i)] = sel[i];
  uint32_t mask[SPL];
  float total[SPL];
  uint32_t same_cnt = 0;                                 // over all of the lane's subsets
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const uint32_t sub = (blockIdx.x * SPL + s) * 256 + tid;
    mask[s] = sub < n_sub ? unrank_device(E, r, sub) : 0u;   // idle: empty pattern, selection index 1, not counted
    total[s] = 0.f;
  }
  const int64_t t_begin = (int64_t)blockIdx.y * tok_tile;
  const int64_t t_end = t_begin + tok_tile < T ? t_begin + tok_tile : T;
  int buf = 0;
  for (int64_t g0 = t_begin; g0 < t_end; g0 += LUT_TG, buf ^= 1) {
    const int ntok = (int)(t_end - g0 < LUT_TG ? t_end - g0 : LUT_TG);
    {
      const uint32_t* src = nibtab + (g0 >> 1) * NT;       // g0 is even
      for (int i = tid; i < ((ntok + 1) >> 1) * NT; i += 256) s_nib[buf][i] = src[i];
    }
    // the group's selection errors: ntok x n_combo consecutive floats
    {
      const float* src = qtab + g0 * n_combo;
      for (int i = tid; i < ntok * n_combo; i += 256) s_q[buf][i] = src[i];
    }
    __syncthreads();      // (also covers s_sel on the first pass; the other buffer is still being read by nobody:
                          //  every thread finished its look-ups in it before it arrived at the previous barrier)
    for (int tk = 0; tk < ntok; tk += 2) {
      const uint32_t* nib = s_nib[buf] + (tk >> 1) * NT;
      const float* qrow = s_q[buf] + tk * n_combo;
      const bool pair = tk + 1 < ntok;                   // the group's last token may stand alone
#pragma unroll
      for (int s = 0; s < SPL; ++s) {
        uint32_t pat = 0;                                // low half: token tk, high half: token tk + 1
#pragma unroll
        for (int nb = 0; nb < NIB; ++nb) pat |= nib[nb * 16 + ((mask[s] >> (4 * nb)) & 15u)];
        const uint32_t si0 = s_sel[lut_swizzle(pat & 0xffffu)];
        total[s] += qrow[si0];
        same_cnt += si0 == 0 ? 1u : 0u;
        if (pair) {
          const uint32_t si1 = s_sel[lut_swizzle(pat >> 16)];
          total[s] += qrow[n_combo + si1];
          same_cnt += si1 == 0 ? 1u : 0u;
        }
        // about 32 look-ups in flight at a time: more only costs registers
        if ((s + 1) % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < SPL; ++s) {
    const uint32_t sub = (blockIdx.x * SPL + s) * 256 + tid;
    if (sub < n_sub) {
      partial[(int64_t)blockIdx.y * n_sub + sub] = total[s];
      partial_cnt[(int64_t)blockIdx.y * n_sub + sub] = (s == 0 && count_same) ? same_cnt : 0u;   // only the sum is used
    }
  }
}

// ------------------------------------------------------------------ scoring through tables that never leave the LDS
// Up to 16 experts.  A workgroup owns a tile of tokens and ALL subsets; per group of `tg` tokens it
//   1. evaluates the error of every selection: U = G d for 64 selections of a token on v_mfma_f32_16x16x4_f32 (fp32 products and
//      sums), then d^T U.  A lane holds VP = ceil(CAP / 4) positions of one selection of each 16; the matrix instruction's
//      operand and result layouts agree on them, and sums over positions are three row swaps per 64 selections;
//   2. spreads the errors over all 2^nb patterns of kept rank positions (a thread writes the same patterns for every
//      token: their selection indices stay in registers), so that
//   3. a (subset, token) pair is ONE look-up: pattern -> error.
// The pattern of a subset is that of its kept experts among the first eight (low) plus that of its kept experts among the
// rest (high).  In lexicographic order the subsets with one low part are neighbours, ordered by their high part; a lane
// takes SPL neighbours, so that it looks up its low pattern once per token and reads SPL consecutive high ones.  A word
// holds the patterns of two tokens, as byte offsets of their entries.
// Where pattern `pat` of a token is kept: its bits from 5 up are folded onto the five that choose the bank, by columns of
// which no three cancel.  The patterns of a wavefront differ in the positions of the few experts that vary among its lanes,
// any of the n_act: 2.0 different addresses in the fullest bank of 32 lanes, 9.3 without the fold.  The fold is linear over
// XOR, and low and high patterns share no bit: the tables hold folded ones, the look-up XORs two of them.
// What bounds it: no single unit.  E 16, k 4, 65536 tokens, r = 8 (495 selections, 12870 subsets): 384 us, where the tables in
// global memory and their look-ups took 234 + 664; r = 12 (70, 1820): 82 us, 42 + 109 before; 33 tokens of r = 8, the whole
// call: 150 -> 57 us.  Left out one at a time, of the 384: phase 1 140 us, phase 2 64, phase 3 57, the pattern tables 19; about
// 45 are set-up and the partial sums.  Phase 1 by fp32 FMAs with the record in scalar registers took 230 VALU operations
// per 64 selections and token where it takes 100 and 12 matrix instructions now, records in the LDS.
constexpr int FUSED_MAX_E = 16, FUSED_PER_THREAD = 4;        // patterns per thread and pass of phase 2
__device__ __forceinline__ uint32_t fold_column(int j) {     // of rank position j
  constexpr uint32_t fold[7] = {7, 11, 13, 14, 19, 21, 22};
  uint32_t c = 1u << j;
#pragma unroll
  for (int i = 0; i < 7; ++i) c ^= j == 5 + i ? fold[i] : 0u;
  return c;
}
// A token pair's pattern tables: 256 low masks, then the high masks by their number of experts, each number from an even place
// on (8-byte reads), with room for the last lane to read past the end.
constexpr int FUSED_LOW = 8, FUSED_TAB = 256 + 256 + 32, FUSED_ERRORS = 1024;   // (errors of a group: tokens x whole chunks of 64)
__host__ __device__ constexpr int fused_pattern_bits(int n_act) { return n_act < 6 ? 6 : n_act; }   // tables of whole wavefronts

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// Rows (16 lanes) r of four values a, b, c, d, added over r: row g of the result is the sum of value g.
__device__ __forceinline__ float rows_to_sums(float a, float b, float c, float d) {
  const u32x2 ab = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const u32x2 cd = __builtin_amdgcn_permlane16_swap(__float_as_uint(c), __float_as_uint(d), false, false);
  const float x = __uint_as_float(ab[0]) + __uint_as_float(ab[1]), y = __uint_as_float(cd[0]) + __uint_as_float(cd[1]);
  const u32x2 xy = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(xy[0]) + __uint_as_float(xy[1]);
}
// v[g] = row g of x, in every row
__device__ __forceinline__ void rows_to_all(float x, float (&v)[4]) {
  const u32x2 h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const u32x2 w = __builtin_amdgcn_permlane16_swap(h[i], h[i], false, false);
    v[2 * i] = __uint_as_float(w[0]);
    v[2 * i + 1] = __uint_as_float(w[1]);
  }
}

// The error of one selection whose logits all lie far below the token's maximum: Eq. 1 relative to the largest SELECTED one
// (see score_kernel).  Rare, and written to need few registers.
template <int CAP>
__device__ __forceinline__ float far_selection_error(const float* R, uint32_t bits) {
  const float m = R[CAP + __ffs(bits) - 1];
  float sum = 0.f, q = 0.f;
#pragma unroll 1
  for (int j = 0; j < CAP; ++j) sum += (bits >> j) & 1u ? __expf(R[CAP + j] - m) : 0.f;
  const float inv = __builtin_amdgcn_rcpf(sum);
  const float* g = R + 3 * CAP;
#pragma unroll 1
  for (int i = 0; i < CAP; ++i) {
    float u = 0.f, di = 0.f;
#pragma unroll 1
    for (int j = i; j < CAP; ++j) {
      const float d = fmaf((bits >> j) & 1u ? __expf(R[CAP + j] - m) : 0.f, inv, -R[2 * CAP + j]);
      if (j == i) di = d;
      u = fmaf(*g++, d, u);
    }
    q = fmaf(di, u, q);
  }
  return q;
}

// (lo or hi half of a) ^ (the same half of b)
template <int HALF>
__device__ __forceinline__ uint32_t xor_half(uint32_t a, uint32_t b) {
  uint32_t d;
  if constexpr (HALF == 0)
    asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_0" : "=v"(d) : "v"(a), "v"(b));
  else
    asm("v_xor_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
typedef __attribute__((address_space(3))) const float* lds_float;

template <int CAP, int SPL>
__global__ __launch_bounds__(1024, 8) void fused_score_lut_kernel(const float* __restrict__ rec_all, int64_t T, int tok_tile, int E,
                                                               int r, int kk, int kfull, int n_act, int n_combo,
                                                               uint32_t n_sub, int tg, float* __restrict__ partial,
                                                               unsigned long long* __restrict__ unaffected) {
  constexpr int RS = rec_size(CAP), VP = (CAP + 3) / 4;
  const int eh = E - FUSED_LOW, nb = fused_pattern_bits(n_act), chunks = (n_combo + 63) >> 6;
  extern __shared__ uint32_t smem[];                                   // (the only LDS of the kernel: at address 0)
  float* const ptab = (float*)smem;                                    // tg x 2^nb
  float* const s_q = ptab + (tg << nb);                                // tg x chunks x 64
  uint32_t* const s_mine = (uint32_t*)(s_q + FUSED_ERRORS);            // a word per thread
  uint16_t* const s_bits = (uint16_t*)(s_mine + 1024);                 // chunks x 64: selections
  uint16_t* const s_selbits = s_bits + LUT_MAX_COMBO;                  // the same by lane
  uint16_t* const s_hpos = s_selbits + LUT_MAX_COMBO;                  // 2^eh
  uint2* const s_off = (uint2*)(s_hpos + 256);                         // a wavefront's places in a record
  float* const s_rec = (float*)(s_off + 64);                           // 2 x tg x RS: records of this and the next group
  uint32_t* const s_tab = (uint32_t*)(s_rec + 2 * tg * RS);            // 2 x tg / 2 x FUSED_TAB
  const int tid = threadIdx.x, threads = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = threads >> 6;
  const int64_t t_begin = (int64_t)blockIdx.x * tok_tile;
  const int count = (int)(T - t_begin < tok_tile ? T - t_begin : tok_tile);    // tokens of this workgroup
  const float* const rec = rec_all + t_begin * RS;

  // records of the group from token g0 on: a quad per thread (tg RS <= 4 x 256)
  const bool fetching = 4 * tid < tg * RS;
  auto fetch = [&](int g0) {
    uint32_t at = 16u * (uint32_t)tid;
    asm volatile("" : "+v"(at));
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (fetching && (int)at < 4 * (count - g0) * RS) v = *(const float4*)((const char*)(rec + (int64_t)g0 * RS) + at);
    return v;
  };
  if (fetching) ((float4*)s_rec)[tid] = fetch(0);

  // ---- set-up.  In the place of the pattern tables: the binomials, the walk of four rank positions at a time, and for every
  // mask of eight experts its place among those of as many experts and the first subset with it as low part.  Every chain of
  // dependent look-ups here is short: the workgroups of a launch start together, and all wait for it.
  uint16_t* const s_binom = (uint16_t*)ptab;                           // 17 x 17
  uint32_t* const s_walk = smem + 160;                                 // [position / 4][experts still to find][their pattern]
  uint8_t* const s_lowmask = (uint8_t*)(s_tab + tg * FUSED_TAB);       // place -> low mask
  uint16_t* const s_first = (uint16_t*)(s_lowmask + 256);              // low mask -> subset
  for (int i = tid; i < 17 * 17; i += threads) s_binom[i] = (uint16_t)c_binom.v[i / 17][i % 17];
  for (int i = tid; i < tg * FUSED_TAB; i += threads) s_tab[i] = 0u;
  for (int c = n_combo + tid; c < chunks * 64; c += threads) s_bits[c] = (uint16_t)((1u << kk) - 1u);   // idle lanes: selection 0
  __syncthreads();
  auto binom = [&](int n, int k) { return (uint32_t)s_binom[n * 17 + k]; };
  // steps of the lexicographic rank: an element not taken, with k still to come among n - 1 further ones, skips C(n - 1, k - 1)
  auto skipped = [&](bool taken, int n, int k) { return taken || k <= 0 ? 0u : binom(n - 1, k - 1); };
  const int walks = (n_act + 3) >> 2;
  for (int i = tid; i < walks * (kk + 1) * 16; i += threads) {
    const int from = 4 * (i / ((kk + 1) * 16));
    int k = (i >> 4) % (kk + 1);
    uint32_t idx = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (from + e < n_act) {
        const bool taken = (i >> e) & 1;
        idx += skipped(taken, n_act - from - e, k);
        k -= taken && k > 0;
      }
    s_walk[i] = idx | (uint32_t)k << 16;
  }
  if (tid < 256) {
    const int m = tid, count8 = __popc((uint32_t)m);
    int kl = count8, kh = count8, kr = r;
    uint32_t low = 0, high = 0, begin = 0, low_place = 0, high_place = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool taken = (m >> e) & 1;
      low += skipped(taken, 8 - e, kl);
      if (e < eh) high += skipped(taken, eh - e, kh);
      begin += skipped(taken, E - e, kr);
      kl -= taken;
      kh -= taken;
      kr -= taken;
      low_place += e < count8 ? binom(8, e) : 0u;
      high_place += e < count8 && e <= eh ? (binom(eh, e) + 1u) & ~1u : 0u;
    }
    s_lowmask[low_place + low] = (uint8_t)m;
    s_first[m] = (uint16_t)begin;                        // (meaningless, and never asked for, with more than r experts)
    if (m < (1 << eh)) s_hpos[m] = (uint16_t)(high_place + high);
  }
  // this lane's subsets: h experts of the high part, entry q of those
  int lanes = 0, mine = -1, q = 0, place = 0;
  {
    int at = 0;
#pragma unroll
    for (int h = 0; h <= FUSED_MAX_E - FUSED_LOW; ++h) {
      const int a = h <= r ? r - h : FUSED_LOW + 1, nh = (int)c_binom.v[eh][h];     // (more of a half than it has: 0 ways)
      const int here = (int)c_binom.v[FUSED_LOW][a] * ((nh + SPL - 1) / SPL);
      if (tid >= lanes && tid < lanes + here) { mine = h; q = tid - lanes; place = at; }
      lanes += here;
      at += (nh + 1) & ~1;
    }
  }
  const bool scoring = wave * 64 < lanes;
  __syncthreads();
  uint32_t lowm = 0;                                     // low part
  int hoff = 0;                                          // place of the first high part
  {
    uint32_t word = 0;                                   // first subset, how many
    if (mine >= 0) {
      const int a = r - mine, nl = (int)binom(FUSED_LOW, a), nh = (int)binom(eh, mine);
      const int seg = (int)(((float)q + 0.5f) * __builtin_amdgcn_rcpf((float)nl));   // q / nl: below 1024 / 70, exact
      uint32_t low_place = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) low_place += e < a ? binom(8, e) : 0u;
      lowm = s_lowmask[low_place + (uint32_t)(q - seg * nl)];
      hoff = place + seg * SPL;
      const int left = nh - seg * SPL;
      word = ((uint32_t)s_first[lowm] + (uint32_t)(seg * SPL)) | (uint32_t)(left < SPL ? left : SPL) << 16;
    }
    s_mine[tid] = word;                                  // not needed before the end
  }
  // this thread's patterns: byte offsets of their selections' errors
  uint32_t sel[FUSED_PER_THREAD];
#pragma unroll
  for (int n = 0; n < FUSED_PER_THREAD; ++n) {
    uint32_t pat = (uint32_t)(tid + n * threads) & ((1u << nb) - 1u), idx = 0;   // bits from 5 up lie where they are
    const uint32_t high = pat >> 5;
    constexpr uint32_t fold[7] = {7, 11, 13, 14, 19, 21, 22};
#pragma unroll
    for (int j = 0; j < 7; ++j) pat ^= (uint32_t)__builtin_amdgcn_sbfe((int)high, j, 1) & fold[j];
    int k = kk;
#pragma unroll
    for (int w = 0; w < 3; ++w)
      if (w < walks) {
        const uint32_t step = s_walk[(w * (kk + 1) + k) * 16 + ((pat >> (4 * w)) & 15u)];
        idx += step & 0xffffu;
        k = (int)(step >> 16);
      }
    if (k == 0 && __popc(pat) == kk && pat < (1u << n_act)) s_bits[idx] = (uint16_t)pat;
    sel[n] = 4u * (k == 0 ? idx : (n_combo > 1 ? 1u : 0u));   // too few bits: no subset has this pattern
  }
  // where a lane's matrix row (a place for each of VP columns) and columns lie in a record, in bytes; beyond CAP or below the
  // diagonal: the record's last word, which is 0
  if (tid < 64) {
    const int row = tid >> 4, slot = tid & 15, pr = VP * (slot >> 2) + (slot & 3);
    uint16_t off[4] = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < VP; ++v) {
      const int j = VP * row + v;
      const bool upper = j < CAP && (slot & 3) < VP && pr <= j;
      off[v] = (uint16_t)(4 * (upper ? 3 * CAP + pr * CAP - pr * (pr - 1) / 2 + j - pr : RS - 1));
    }
    s_off[tid] = make_uint2(off[0] | (uint32_t)off[1] << 16, off[2]);
  }
  __syncthreads();
  for (int c = tid; c < chunks * 64; c += threads) {
    // for this place's lane: bit g VP + v = position VP (lane / 16) + v of selection 16 g + lane % 16 of the 64
    uint32_t word = 0;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      word |= (((uint32_t)s_bits[(c & ~63) + 16 * g + (c & 15)] >> (VP * ((c >> 4) & 3))) & ((1u << VP) - 1u)) << (g * VP);
    s_selbits[c] = (uint16_t)word;
  }
  float total[SPL];
#pragma unroll
  for (int s = 0; s < SPL; ++s) total[s] = 0.f;
  // Pattern tables of the token pairs of the group from token g0 on, a wavefront per pair from the last one down (the last
  // may have no subsets): lane = (low or high half, nibble of it, value), then the masks of 64 lanes at a time.
  auto build_tables = [&](int ntok, const float* records, uint32_t* tabs) {
#pragma unroll 1
    for (int pr = waves - 1 - wave; 2 * pr < ntok; pr += waves) {
      int lane = tid & 63, active = n_act;               // nothing derived from these is worth a register across the loop
      asm volatile("" : "+v"(lane), "+s"(active));
      const uint32_t m = (uint32_t)(lane & 15) << (4 * (lane >> 4));
      uint32_t ordw[2][VP], word = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int w = 0; w < VP; ++w)
          ordw[h][w] = __builtin_amdgcn_readfirstlane(__float_as_int(records[(2 * pr + h) * RS + rec_order_off(CAP) + w]));
#pragma unroll
      for (int j = 0; j < CAP; ++j) {
        const uint32_t column = j < active ? fold_column(j) << 2 : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t e = (ordw[h][j >> 2] >> (8 * (j & 3))) & 0x1fu;
          word ^= (column << (16 * h)) & (uint32_t)__builtin_amdgcn_sbfe((int)m, e, 1);
        }
      }
      uint32_t* tab = tabs + pr * FUSED_TAB;
      const uint32_t l0 = __shfl(word, lane & 15), h0 = __shfl(word, 32 + (lane & 15));
#pragma unroll
      for (int c = 0; c < 256; c += 64) tab[c + lane] = l0 ^ __shfl(word, 16 + ((c + lane) >> 4));
#pragma unroll
      for (int c = 0; c < 256; c += 64) {
        const uint32_t pat = h0 ^ __shfl(word, 48 + ((c + lane) >> 4));   // (every lane takes part)
        if (c + lane < (1 << eh)) tab[256 + s_hpos[c + lane]] = pat;
      }
    }
  };
  // Phase 1 for the ntok tokens of a group.
  auto errors = [&](int ntok, const float* records) {
    int lane = tid & 63;
    asm volatile("" : "+v"(lane));
    const uint2 off = s_off[lane];
    for (int job = wave; job < ((ntok + 1) & ~1) * chunks; job += waves) {
      const int tk = job / chunks, chunk = job - tk * chunks;
      float q = 0.f;                                   // a group's last token may have no partner: errors of 0
      if (tk < ntok) {
        const float* R = records + tk * RS;
        float ga[VP], ex[VP], aw[VP];
#pragma unroll
        for (int v = 0; v < VP; ++v) {
          const int j = VP * (lane >> 4) + v;
          const bool in = 4 * VP == CAP || j < CAP;
          ga[v] = *(const float*)((const char*)R + (v == 0 ? off.x & 0xffffu : v == 1 ? off.x >> 16 : off.y));
          ex[v] = R[in ? j : RS - 1];
          aw[v] = R[in ? 2 * CAP + j : RS - 1];
        }
        const int word = s_selbits[chunk * 64 + lane];
        float d[4][VP], part[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
#pragma unroll
          for (int v = 0; v < VP; ++v) {
            d[g][v] = __uint_as_float(__float_as_uint(ex[v]) & (uint32_t)__builtin_amdgcn_sbfe(word, g * VP + v, 1));
            part[g] = v == 0 ? d[g][v] : part[g] + d[g][v];
          }
        }
        const float sum = rows_to_sums(part[0], part[1], part[2], part[3]);
        float inv[4];
        rows_to_all(__builtin_amdgcn_rcpf(sum), inv);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int v = 0; v < VP; ++v) d[g][v] = fmaf(d[g][v], inv[g], -aw[v]);
#pragma unroll
          for (int v = 0; v < VP; ++v) u = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[v], d[g][v], u, 0, 0, 0);
          part[g] = d[g][0] * u[0];
#pragma unroll
          for (int v = 1; v < VP; ++v) part[g] = fmaf(d[g][v], u[v], part[g]);
        }
        q = rows_to_sums(part[0], part[1], part[2], part[3]);
        const int c = chunk * 64 + lane;
        if (__any(sum < 1e-30f)) {
          if (sum < 1e-30f) q = far_selection_error<CAP>(R, s_bits[c]);
        }
        if (kk == kfull && c == 0) q = 0.f;
      }
      s_q[job * 64 + lane] = q;
    }
  };
  // Phase 3.
  auto look_up = [&](int pairs, const uint32_t* tabs) {
    for (int pr = 0; pr < pairs; ++pr) {
      const uint32_t* tab = tabs + pr * FUSED_TAB;
      const uint32_t at = (uint32_t)(8 * pr) << nb;                   // address of the pair's first table
      const uint32_t pl = tab[lowm] ^ (at | (at + (4u << nb)) << 16);
      const uint2* ph = (const uint2*)(tab + 256 + hoff);
#pragma unroll
      for (int s = 0; s < SPL; s += 2) {
        const uint2 h = ph[s >> 1];
        total[s] += *(lds_float)(uintptr_t)xor_half<0>(pl, h.x);
        total[s] += *(lds_float)(uintptr_t)xor_half<1>(pl, h.x);
        total[s + 1] += *(lds_float)(uintptr_t)xor_half<0>(pl, h.y);
        total[s + 1] += *(lds_float)(uintptr_t)xor_half<1>(pl, h.y);
      }
    }
  };

  // Between two barriers: phase 2 of a group; then its phase 3 and phase 1 of the next one.  Half of a SIMD's wavefronts take
  // these two in the other order, so that look-ups (LDS) and errors (VALU, matrix unit) run beside each other.
  const bool errors_first = (wave >> 2) & 1;
  int buf = 1;                                           // of records and pattern tables of the group that is looked up
  for (int g0 = -tg; g0 < count; g0 += tg, buf ^= 1) {
    const int here = g0 < 0 ? 0 : count - g0 < tg ? count - g0 : tg, pairs = (here + 1) >> 1;
    const int left = count - g0 - tg, after = left < tg ? left : tg;
    {
      uint32_t at = 4u * (uint32_t)tid;
      asm volatile("" : "+v"(at));
      const int end = (2 * pairs) << nb;
      for (int f = 0; f < end; f += FUSED_PER_THREAD * threads) {
        float e[FUSED_PER_THREAD];
#pragma unroll
        for (int n = 0; n < FUSED_PER_THREAD; ++n) {     // (beyond the group's tokens: read within s_q, not written)
          int tk = (f + n * threads + wave * 64) >> nb;
          tk = tk < tg ? tk : tg - 1;
          e[n] = *(const float*)((const char*)s_q + ((uint32_t)(tk * chunks * 256) + sel[n]));
        }
#pragma unroll
        for (int n = 0; n < FUSED_PER_THREAD; ++n)
          if (f + n * threads + wave * 64 < end) *(float*)((char*)ptab + ((uint32_t)(4 * (f + n * threads)) + at)) = e[n];
      }
    }
    __syncthreads();
    const float4 next = fetch(g0 + 2 * tg);
    const float* const records = s_rec + (buf ^ 1) * tg * RS;
    if (after > 0) build_tables(after, records, s_tab + (buf ^ 1) * (tg / 2) * FUSED_TAB);
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      if (errors_first == (half == 0)) {
        if (after > 0) errors(after, records);
      } else if (scoring) {
        look_up(pairs, s_tab + buf * (tg / 2) * FUSED_TAB);
      }
    }
    if (fetching) ((float4*)(s_rec + buf * tg * RS))[tid] = next;      // last read before the barrier before
    __syncthreads();
  }
  {
    int me = tid;
    asm volatile("" : "+v"(me));
    const uint32_t word = s_mine[me];                    // this thread's own word
    float* const out = partial + (int64_t)blockIdx.x * n_sub + (word & 0xffffu);
    const int live = (int)(word >> 16);
    if (live == SPL) {
      __builtin_memcpy(out, total, sizeof(total));       // 16 bytes a store, at any place
    } else {
#pragma unroll
      for (int s = 0; s < SPL; ++s)
        if (s < live) out[s] = total[s];
    }
  }
  if (unaffected && kk == kfull) {
    // pairs whose selection is the full layer's: the subsets that keep the token's first k experts
    unsigned long long same = 0;
    for (int i = tid; i < count; i += threads) {
      const uint32_t* const ordw = (const uint32_t*)(rec + (int64_t)i * RS + rec_order_off(CAP));
      uint32_t top = 0;
      for (int j = 0; j < kk; ++j) top |= 1u << ((ordw[j >> 2] >> (8 * (j & 3))) & 0x1fu);
      const int distinct = __popc(top);
      same += c_binom.v[E - distinct][r - distinct];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) same += __shfl_xor(same, off, 64);
    if (same && (tid & 63) == 0) atomicAdd(unaffected, same);          // integer: order does not matter
  }
}

// Lanes of the fused scorer with spl subsets each (E > FUSED_LOW).
int fused_lanes(int E, int r, int spl) {
  int64_t lanes = 0;
  for (int h = 0; h <= E - FUSED_LOW && h <= r; ++h)
    if (r - h <= FUSED_LOW) lanes += binomial(FUSED_LOW, r - h) * ceil_div(binomial(E - FUSED_LOW, h), spl);
  return (int)lanes;
}
size_t fused_lds(int n_act, int rec_floats, int tg) {
  return (((size_t)tg << fused_pattern_bits(n_act)) + FUSED_ERRORS + 1024 + LUT_MAX_COMBO + 128 + 128 + tg * (2 * rec_floats + FUSED_TAB)) * 4 +
         256 + 512;
}

// ------------------------------------------------------------------ reduce + argmin
__global__ __launch_bounds__(256) void zero_i64_kernel(unsigned long long* p) { *p = 0ull; }

// Partial sums to be reduced: those of one r, or of several in one launch.
struct ReduceJob {
  const float* partial; const uint32_t* partial_cnt;      // partial_cnt NULL: counted elsewhere
  int64_t n_tiles;
  uint32_t n_sub, first_block;                            // first_block: of reduce_kernel
  int S, r;                                               // S: reduce_one_kernel's subsets at a time
  float* loss; unsigned long long* unaffected; int32_t* argmin; uint32_t* argmin_mask;
};
struct ReduceSet { int n; ReduceJob job[RECORD_SETS]; };

// A workgroup adds the partial sums of SUBS neighbouring subsets: thread (strand, j) adds tiles strand,
// strand + 256 / SUBS, ... of subset j in fp64, then a tree over the strands; the order depends on nothing but
// the tile count and SUBS.  SUBS = 1 suits a handful of subsets; with thousands, SUBS = 32 reads the partial
// sums (subset index fastest) in 128-byte runs.
template <int SUBS>
__global__ __launch_bounds__(256) void reduce_kernel(ReduceSet set) {
  int which = 0;
  while (which + 1 < set.n && blockIdx.x >= set.job[which + 1].first_block) ++which;
  const ReduceJob& job = set.job[which];
  const float* __restrict__ const partial = job.partial;
  const uint32_t* __restrict__ const partial_cnt = job.partial_cnt;
  const int64_t n_tiles = job.n_tiles;
  const uint32_t n_sub = job.n_sub;
  constexpr int STRANDS = 256 / SUBS;
  __shared__ double ss[256];
  __shared__ unsigned long long sc[256];
  const int j = threadIdx.x % SUBS, strand = threadIdx.x / SUBS;
  const uint32_t sub = (blockIdx.x - job.first_block) * SUBS + j;
  double s = 0.0;
  unsigned long long c = 0;
  if (sub < n_sub)
#pragma unroll 8
    for (int64_t i = strand; i < n_tiles; i += STRANDS) {
      s += (double)partial[i * n_sub + sub];
      if (partial_cnt) c += partial_cnt[i * n_sub + sub];
    }
  ss[threadIdx.x] = s;
  sc[threadIdx.x] = c;
  __syncthreads();
  for (int off = STRANDS / 2; off >= 1; off >>= 1) {
    if (strand < off) {
      ss[threadIdx.x] += ss[threadIdx.x + off * SUBS];
      sc[threadIdx.x] += sc[threadIdx.x + off * SUBS];
    }
    __syncthreads();
  }
  if (strand == 0 && sub < n_sub) {
    job.loss[sub] = (float)ss[threadIdx.x];
    if (job.unaffected && sc[threadIdx.x]) atomicAdd(job.unaffected, sc[threadIdx.x]);   // integer: order does not matter
  }
}

__global__ __launch_bounds__(1024) void argmin_kernel(ReduceSet set, int E) {
  const ReduceJob& job = set.job[blockIdx.x];
  const float* __restrict__ const loss = job.loss;
  const uint32_t n_sub = job.n_sub;
  __shared__ float sv[1024];
  __shared__ uint32_t si[1024];
  float best = INFINITY;
  uint32_t bi = 0xffffffffu;
  for (uint32_t i = threadIdx.x; i < n_sub; i += 1024) {
    const float v = loss[i];
    if (v < best || bi == 0xffffffffu) { best = v; bi = i; }   // ascending i: first minimum wins
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int off = 512; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) {
      const float v = sv[threadIdx.x + off];
      const uint32_t i = si[threadIdx.x + off];
      const float mv = sv[threadIdx.x];
      const uint32_t mi = si[threadIdx.x];
      if (i != 0xffffffffu && (mi == 0xffffffffu || v < mv || (v == mv && i < mi))) {
        sv[threadIdx.x] = v;
        si[threadIdx.x] = i;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const uint32_t i = si[0] == 0xffffffffu ? 0u : si[0];
    *job.argmin = (int32_t)i;
    *job.argmin_mask = unrank_device(E, job.r, i);
  }
}

// reduce and argmin in one workgroup per r, for few partial sums: thread (strand, j) adds tiles strand, strand + strands, ... of
// subsets j, j + S, ... in fp64 (S = the power of two from n_sub up, at most 1024), a tree over the strands, then the
// workgroup's argmin.  Also writes the count of unaffected pairs, so that nothing has to be cleared first.
__global__ __launch_bounds__(1024) void reduce_one_kernel(ReduceSet set, int E) {
  const ReduceJob& job = set.job[blockIdx.x];
  const float* __restrict__ const partial = job.partial;
  const uint32_t* __restrict__ const partial_cnt = job.partial_cnt;
  const int n_tiles = (int)job.n_tiles, S = job.S;
  const uint32_t n_sub = job.n_sub;
  __shared__ double ss[1024];
  __shared__ unsigned long long sc[1024];
  __shared__ float sv[1024];
  __shared__ uint32_t si[1024];
  const int j = threadIdx.x & (S - 1), strand = threadIdx.x / S, strands = 1024 / S;
  unsigned long long c = 0;
  float best = INFINITY;
  uint32_t bi = 0xffffffffu;
  for (uint32_t s0 = 0; s0 < n_sub; s0 += S) {
    const uint32_t sub = s0 + j;
    double s = 0.0;
    if (sub < n_sub)
#pragma unroll 4
      for (int i = strand; i < n_tiles; i += strands) {
        s += (double)partial[(int64_t)i * n_sub + sub];
        if (partial_cnt) c += partial_cnt[(int64_t)i * n_sub + sub];
      }
    ss[threadIdx.x] = s;
    __syncthreads();
    for (int off = strands >> 1; off >= 1; off >>= 1) {
      if (strand < off) ss[threadIdx.x] += ss[threadIdx.x + off * S];
      __syncthreads();
    }
    if (strand == 0 && sub < n_sub) {
      const float v = (float)ss[threadIdx.x];
      job.loss[sub] = v;
      if (v < best || bi == 0xffffffffu) { best = v; bi = sub; }   // ascending: first minimum wins
    }
  }
  sc[threadIdx.x] = c;
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int off = 512; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) {
      sc[threadIdx.x] += sc[threadIdx.x + off];
      const float v = sv[threadIdx.x + off];
      const uint32_t i = si[threadIdx.x + off];
      const float mv = sv[threadIdx.x];
      const uint32_t mi = si[threadIdx.x];
      if (i != 0xffffffffu && (mi == 0xffffffffu || v < mv || (v == mv && i < mi))) {
        sv[threadIdx.x] = v;
        si[threadIdx.x] = i;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (job.unaffected) *job.unaffected = sc[0];
    const uint32_t i = si[0] == 0xffffffffu ? 0u : si[0];
    *job.argmin = (int32_t)i;
    *job.argmin_mask = unrank_device(E, job.r, i);
  }
}

// Lanes per scoring workgroup: one lane per subset, whole wavefronts, at most four of them.
int score_threads(int64_t n_sub) {
  return n_sub >= 256 ? 256 : (int)((n_sub + 63) / 64) * 64;
}

int capacity_for(int n_act) {
  const int caps[] = {2, 4, 6, 8, 12, 16, 32};
  for (int c : caps)
    if (n_act <= c) return c;
  return -1;
}

}  // namespace

int plan_enumerate(int64_t T, int E, int H, int k, int r, EnumPlan* p) {
  if (k < 1 || k > E) return fail(MOEP_EINVAL, "prune_enumerate: k=%d out of range [1, E=%d]", k, E);
  if (r < 1 || r > E) return fail(MOEP_EINVAL, "prune_enumerate: r=%d out of range [1, E=%d]", r, E);
  p->T = T; p->E = E; p->H = H; p->k = k; p->r = r;
  p->kk = k < r ? k : r;
  const int n_act = p->kk + E - r;
  p->n_act = n_act < E ? n_act : E;
  p->n_sub = binomial(E, r);
  if (p->n_sub > ((int64_t)1 << 24))
    return fail(MOEP_EUNSUPPORTED, "prune_enumerate: C(%d,%d) = %lld subsets exceeds 2^24", E, r, (long long)p->n_sub);
  const int cap = capacity_for(p->n_act);
  p->rec_floats = rec_size(cap);
  // With many subsets and few possible selections per token, score through per-token selection tables.
  const int64_t n_combo = binomial(p->n_act, p->kk);
  p->n_combo = (int)(n_combo < (1 << 20) ? n_combo : (1 << 20));
  p->use_lut = p->n_sub >= 512 && p->n_act <= LUT_MAX_ACT && n_combo <= LUT_MAX_COMBO;
  const bool fused = p->use_lut && E <= FUSED_MAX_E;
  if (p->use_lut) {
    // Up to 16 experts the fused scorer has a shape of its own, below; the shape here then only gives the size of the
    // workspace, which is the one that callers reserved for tables in memory and that the limit of prune_enumerate_static goes
    // by.  Of the room behind the records it takes what its partial sums need; sizing it by those alone would make some sizes
    // larger (16 experts, r = 7, one expert per token: up to 70000 tokens) and so refuse batches that were accepted.
    // Subsets per lane there: 8 or 17, whichever leaves fewer idle slots in the last workgroup of 256 lanes.
    const bool wide = fused && ceil_div(p->n_sub, 256 * 17) * 17 < ceil_div(p->n_sub, 256 * LUT_SPL) * LUT_SPL;
    // Workgroups of equal length, about as many as a 256-CU part holds at once (three per CU by their LDS): tiles
    // of whole token groups, 32 to 1024 tokens.
    const int64_t sub_blocks = ceil_div(p->n_sub, 256 * (wide ? 17 : LUT_SPL));
    const int64_t want_tiles = sub_blocks < 768 ? 768 / sub_blocks : 1;
    int64_t tile = ceil_div(ceil_div(T, want_tiles), LUT_TG) * LUT_TG;
    tile = tile < 32 ? 32 : tile > 1024 ? 1024 : tile;
    p->tok_tile = (int)tile;
  } else {
    // Aim for a few thousand scoring workgroups; tiles of 32..256 tokens.
    const int64_t sub_blocks = ceil_div(p->n_sub, score_threads(p->n_sub));
    int tile = 256;
    while (tile > 32 && sub_blocks * ceil_div(T, tile) < 4096) tile >>= 1;
    p->tok_tile = tile;
  }
  p->n_tok_tiles = ceil_div(T, p->tok_tile);
  if (p->n_tok_tiles > 65535) {                          // the grid's second dimension
    p->tok_tile = (int)(ceil_div(ceil_div(T, 65535), LUT_TG) * LUT_TG);
    p->n_tok_tiles = ceil_div(T, p->tok_tile);
  }
  size_t off = 0;
  p->off_gram = off; off += align256((size_t)T * E * E * sizeof(float));
  p->off_rec = off; off += align256((size_t)T * p->rec_floats * sizeof(float));
  p->off_masks = off;
  p->off_partial = off; off += align256((size_t)p->n_tok_tiles * p->n_sub * sizeof(float));
  p->off_partial_cnt = off; off += align256((size_t)p->n_tok_tiles * p->n_sub * sizeof(uint32_t));
  p->off_qtab = p->off_sel = p->off_selbits = p->off_nib = off;
  if (p->use_lut) {
    p->off_qtab = off; off += align256((size_t)T * p->n_combo * sizeof(float));
    p->off_sel = off; off += align256(((size_t)1 << p->n_act) * sizeof(uint16_t));
    p->off_selbits = off; off += align256((size_t)p->n_combo * sizeof(uint16_t));
    p->off_nib = off; off += align256((size_t)((T + 1) / 2) * ((E + 3) / 4) * 16 * sizeof(uint32_t));
  }
  p->total = off > 0 ? off : 256;
  p->fused_threads = 0;
  if (fused && T > 0) {
    // Subsets per lane: 4 where that takes no more than 1024 lanes, else 14 (12870 subsets: 928 lanes).
    p->fused_spl = fused_lanes(E, r, 4) <= 1024 ? 4 : 14;
    int threads = 256;
    while (threads < fused_lanes(E, r, p->fused_spl) || threads * FUSED_PER_THREAD < (1 << p->n_act)) threads <<= 1;
    // Tokens per barrier: 8, fewer where their tables would keep the compute unit from its workgroups or exceed 64 KB.
    int tg = 8;
    const int chunks = (p->n_combo + 63) / 64, per_cu = threads <= 512 ? 4 : 2;
    while (tg > 2 && (fused_lds(p->n_act, p->rec_floats, tg) > (size_t)(per_cu == 2 ? 64 : 40) * 1024 || tg * chunks * 64 > FUSED_ERRORS)) tg >>= 1;
    p->fused_tg = tg;
    p->fused_lds = fused_lds(p->n_act, p->rec_floats, tg);
    p->fused_threads = threads;
    // One resident round of equal workgroups on 256 compute units, tiles of 8 tokens at least; several rounds where a lane
    // would otherwise add more than 1024 tokens in fp32 (relative error of such sums of positive terms, simulated: 2^20 tokens
    // by 1024 1.1e-8, by 2048 2.3e-8; 2^22 tokens by 1024 0.5e-8, by 8192 7.5e-8).  Their partial sums take the place of the
    // tables and counts of the scorer above.
    int64_t want = 256 * per_cu;
    const int64_t room = (int64_t)((p->off_sel - p->off_partial) / ((size_t)p->n_sub * sizeof(float)));
    want = want < room ? want : room;
    int64_t tile = ceil_div(ceil_div(T, want), tg) * tg;
    tile = tile < 8 ? 8 : tile > 1024 ? 1024 : tile;
    p->tok_tile = (int)tile;
    p->n_tok_tiles = ceil_div(T, tile);
  }
  return MOEP_OK;
}

template <int CAP>
static void launch_score(const EnumPlan& p, const float* rec, float* partial, uint32_t* pcnt,
                         hipStream_t s) {
  const int threads = score_threads(p.n_sub);
  dim3 grid((unsigned)ceil_div(p.n_sub, threads), (unsigned)p.n_tok_tiles);
  // 256 subsets and more: strands only where there are too few workgroups without (1820 subsets of 16 ranks, 5000 tokens:
  // 126 us without, 150 with; 2024 subsets of 23 ranks, 3000 tokens: 391 without, 329 with).
  const int most = threads == 256 && (int64_t)grid.x * grid.y >= 1024 ? 1 : SCORE_STRANDS;
  const int strands = 1024 / threads < most ? 1024 / threads : most;
#define MOEP_SCORE(EXACT, STRANDS)                                                                                     \
  hipLaunchKernelGGL((score_kernel<CAP, EXACT, STRANDS>), grid, dim3(threads, strands), 0, s, rec, p.T, p.tok_tile, p.E, \
                     p.r, p.kk, p.k, p.n_act, (uint32_t)p.n_sub, partial, pcnt)
  if (p.n_act == CAP) {
    if (strands > 1) MOEP_SCORE(true, true);
    else MOEP_SCORE(true, false);
  } else {
    if (strands > 1) MOEP_SCORE(false, true);
    else MOEP_SCORE(false, false);
  }
#undef MOEP_SCORE
}

bool records_by_gram_pass(const EnumPlan* const* plans, int n, int n_rank, bool f32, size_t ws_bytes, RecordPlan* out) {
  const EnumPlan& p0 = *plans[0];
  if (p0.E > 16 || p0.T == 0 || n > RECORD_SETS) return false;
  int weights = 0;
  for (int i = 0; i < n; ++i) weights += record_weight(plans[i]->n_act);
  if (!records_pay(p0.T, n_rank ? n_rank : p0.E, p0.H, f32, n_rank != 0, weights)) return false;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += align256(bytes); return o; };
  for (int i = 0; i < n; ++i) {
    const EnumPlan& p = *plans[i];
    const size_t sums = (size_t)p.n_tok_tiles * p.n_sub * sizeof(float);
    out->rec[i] = take((size_t)p.T * p.rec_floats * sizeof(float));
    out->partial[i] = take(sums);
    out->cnt[i] = take(p.fused_threads ? 0 : sums);
  }
  return off <= ws_bytes;
}

// Whether the Gram kernel can write the records itself: up to 16 experts, rows of whole 16-byte chunks.
static bool gram_writes_records(const EnumPlan& p, const void* Y, moep_dtype dt) {
  return p.E <= 16 && (dt == MOEP_BF16 || (p.H % 4 == 0 && ((uintptr_t)Y & 15) == 0));
}

// G: where the Gram matrices go; recs.n > 0: records instead (the kernels that read word by word and those of more than 16 experts
// write Gram matrices only).
static int launch_gram(const EnumPlan& p, const void* Y, moep_dtype dt, float* G, const RecordArgs& recs,
                       const RankedSource* ranked, hipStream_t s) {
  Timed t("gram", s);
  const unsigned per_tok_blocks = (unsigned)ceil_div(p.T, 4);
  // streaming loads for a Y beyond half a GB
  const bool stream = (double)p.T * (ranked ? ranked->n_rank : p.E) * p.H * 2.0 >= 512.0 * 1024 * 1024;
#define MOEP_GRAM_FORM(EPAD, RANKED, RECORDS, GRID, ...)                                                                  \
  do {                                                                                                                   \
    if (dt != MOEP_BF16)                                                                                                 \
      hipLaunchKernelGGL((gram_kernel<true, EPAD, RANKED, false, RECORDS>), dim3(GRID), dim3(256), 0, s, __VA_ARGS__, recs); \
    else if (stream)                                                                                                     \
      hipLaunchKernelGGL((gram_kernel<false, EPAD, RANKED, true, RECORDS>), dim3(GRID), dim3(256), 0, s, __VA_ARGS__, recs); \
    else                                                                                                                 \
      hipLaunchKernelGGL((gram_kernel<false, EPAD, RANKED, false, RECORDS>), dim3(GRID), dim3(256), 0, s, __VA_ARGS__, recs); \
  } while (0)
#define MOEP_GRAM_LAUNCH(EPAD, RANKED, GRID, ...)                                                                         \
  do {                                                                                                                   \
    if (recs.n > 0) MOEP_GRAM_FORM(EPAD, RANKED, true, GRID, __VA_ARGS__);                                               \
    else MOEP_GRAM_FORM(EPAD, RANKED, false, GRID, __VA_ARGS__);                                                         \
  } while (0)
  // fp32 rows that are not whole 16-byte chunks go through the kernels that read word by word
  const bool by_word = dt != MOEP_BF16 && (p.H % 4 || ((uintptr_t)Y & 15));
  if (by_word && ranked)
    hipLaunchKernelGGL(gram_ranked_f32_kernel, dim3(per_tok_blocks), dim3(256), 0, s, (const float*)Y, ranked->slot_of,
                       ranked->experts, G, p.T, p.E, ranked->n_rank, p.H);
  else if (by_word)
    hipLaunchKernelGGL(gram_f32_kernel, dim3(per_tok_blocks), dim3(256), 0, s, (const float*)Y, G, p.T, p.E, p.H);
  else if (ranked) {
    const int n = ranked->n_rank;
    if (n <= 4)
      MOEP_GRAM_LAUNCH(4, true, (unsigned)ceil_div(p.T, 16), (const uint4*)Y, ranked->slot_of, ranked->experts, G,
                       p.T, p.E, n, p.H);
    else if (n <= 8)
      MOEP_GRAM_LAUNCH(8, true, (unsigned)ceil_div(p.T, 8), (const uint4*)Y, ranked->slot_of, ranked->experts, G,
                       p.T, p.E, n, p.H);
    else
      MOEP_GRAM_LAUNCH(16, true, per_tok_blocks, (const uint4*)Y, ranked->slot_of, ranked->experts, G, p.T, p.E, n,
                       p.H);
  } else if (p.E <= 4) {
    MOEP_GRAM_LAUNCH(4, false, (unsigned)ceil_div(p.T, 16), (const uint4*)Y, nullptr, nullptr, G, p.T, p.E, 0, p.H);
  } else if (p.E <= 8) {
    MOEP_GRAM_LAUNCH(8, false, (unsigned)ceil_div(p.T, 8), (const uint4*)Y, nullptr, nullptr, G, p.T, p.E, 0, p.H);
  } else if (p.E <= 16) {
    MOEP_GRAM_LAUNCH(16, false, per_tok_blocks, (const uint4*)Y, nullptr, nullptr, G, p.T, p.E, 0, p.H);
  } else if (dt == MOEP_BF16) {
    hipLaunchKernelGGL(gram_bf16_32_kernel, dim3(per_tok_blocks), dim3(256), 0, s, (const uint4*)Y, G, p.T, p.E, p.H);
  } else {
    hipLaunchKernelGGL(gram_f32_32_kernel, dim3((unsigned)ceil_div(p.T, 2)), dim3(128), 0, s, (const uint4*)Y, G, p.T, p.E, p.H);
  }
#undef MOEP_GRAM_LAUNCH
#undef MOEP_GRAM_FORM
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

// Partial sums of every subset's error over tiles of tokens, from the records; the tables of the scorer of more than 16 experts
// lie where the plan has them.
static int launch_scores(const EnumPlan& p, const float* rec, float* partial, uint32_t* pcnt, char* ws, int64_t* unaffected,
                         hipStream_t s) {
  const int cap = capacity_for(p.n_act);
  if (p.fused_threads) {
    Timed t("subset_score_tables", s);
#define MOEP_FUSED(C, S)                                                                                               \
  hipLaunchKernelGGL((fused_score_lut_kernel<C, S>), dim3((unsigned)p.n_tok_tiles), dim3(p.fused_threads), p.fused_lds, \
                   s, rec, p.T, p.tok_tile, p.E, p.r, p.kk, p.k, p.n_act, p.n_combo, (uint32_t)p.n_sub, p.fused_tg,  \
                   partial, (unsigned long long*)unaffected)
    switch (cap * 100 + p.fused_spl) {                 // (4 active ranks: 560 subsets, 4 per lane)
      case 404: MOEP_FUSED(4, 4); break;
      case 604: MOEP_FUSED(6, 4); break;
      case 614: MOEP_FUSED(6, 14); break;
      case 804: MOEP_FUSED(8, 4); break;
      case 814: MOEP_FUSED(8, 14); break;
      case 1204: MOEP_FUSED(12, 4); break;
      case 1214: MOEP_FUSED(12, 14); break;
      default: return fail(MOEP_EUNSUPPORTED, "prune_enumerate: no selection table for %d active ranks", p.n_act);
    }
#undef MOEP_FUSED
    MOEP_HIP(hipGetLastError());
  } else if (p.use_lut) {
    Timed t("subset_score_tables", s);
    float* qtab = (float*)(ws + p.off_qtab);
    uint16_t* sel = (uint16_t*)(ws + p.off_sel);
    uint16_t* selbits = (uint16_t*)(ws + p.off_selbits);
    hipLaunchKernelGGL(selidx_kernel, dim3((unsigned)ceil_div((int64_t)1 << p.n_act, 256)), dim3(256), 0, s, p.n_act,
                       p.kk, sel, selbits);
    uint16_t* nibtab = (uint16_t*)(ws + p.off_nib);
    const int nib = (p.E + 3) / 4;
    const dim3 qgrid((unsigned)p.T), qblock(p.n_combo <= 64 ? 64 : 256);
#define MOEP_QTABLE(C, EXACT)                                                                                     \
  hipLaunchKernelGGL((qtable_kernel<C, EXACT>), qgrid, qblock, 0, s, rec, p.kk, p.k, p.n_act, p.n_combo, selbits, qtab, nib, nibtab)
#define MOEP_QTABLE_CASE(C)                                                                                       \
  case C:                                                                                                         \
  if (p.n_act == C) MOEP_QTABLE(C, true);                                                                       \
  else MOEP_QTABLE(C, false);                                                                                   \
  break;
    switch (cap) {
      case 4: MOEP_QTABLE(4, true); break;             // (up to 3 active ranks have fewer than 512 subsets)
      MOEP_QTABLE_CASE(6) MOEP_QTABLE_CASE(8) MOEP_QTABLE_CASE(12)
      default: return fail(MOEP_EUNSUPPORTED, "prune_enumerate: no selection table for %d active ranks", p.n_act);
    }
#undef MOEP_QTABLE_CASE
#undef MOEP_QTABLE
    const dim3 grid((unsigned)ceil_div(p.n_sub, 256 * LUT_SPL), (unsigned)p.n_tok_tiles);
    const bool count_same = p.kk == p.k;
#define MOEP_LUT_LAUNCH(N)                                                                                        \
  hipLaunchKernelGGL((score_lut_kernel<N>), grid, dim3(256), 0, s, qtab, (const uint32_t*)nibtab, sel, p.T, p.tok_tile, p.E,    \
                   p.r, p.n_act, p.n_combo, count_same, (uint32_t)p.n_sub, partial, pcnt)
    switch (nib) {                                     // (up to 16 experts: above)
      case 5: MOEP_LUT_LAUNCH(5); break;
      case 6: MOEP_LUT_LAUNCH(6); break;
      case 7: MOEP_LUT_LAUNCH(7); break;
      case 8: MOEP_LUT_LAUNCH(8); break;
      default: return fail(MOEP_EUNSUPPORTED, "prune_enumerate: no table scorer for %d experts", p.E);
    }
#undef MOEP_LUT_LAUNCH
    MOEP_HIP(hipGetLastError());
  } else {
    Timed t("subset_score", s);
    switch (cap) {
      case 2: launch_score<2>(p, rec, partial, pcnt, s); break;
      case 4: launch_score<4>(p, rec, partial, pcnt, s); break;
      case 6: launch_score<6>(p, rec, partial, pcnt, s); break;
      case 8: launch_score<8>(p, rec, partial, pcnt, s); break;
      case 12: launch_score<12>(p, rec, partial, pcnt, s); break;
      case 16: launch_score<16>(p, rec, partial, pcnt, s); break;
      case 32: launch_score<32>(p, rec, partial, pcnt, s); break;
      default: return fail(MOEP_EUNSUPPORTED, "prune_enumerate: no scorer for %d active ranks", p.n_act);
    }
    MOEP_HIP(hipGetLastError());
  }
  return MOEP_OK;
}

int launch_enumerate_from_gram(const EnumJob& job, const float* logits, const void* Y, moep_dtype dt, char* ws, hipStream_t s,
                               const RankedSource* ranked, bool reuse_gram) {
  const EnumPlan& p = job.plan;
  int64_t* const unaffected = job.unaffected;
  float* G = (float*)(ws + p.off_gram);
  float* rec = (float*)(ws + p.off_rec);
  float* partial = (float*)(ws + p.off_partial);
  uint32_t* pcnt = (uint32_t*)(ws + p.off_partial_cnt);
  const int cap = capacity_for(p.n_act);
  if (p.T > 0) {
    // The Gram matrices do not depend on r: a caller that scores several r on the same logits and Y (and the same
    // workspace: G sits at its start whatever r is) computes them once.
    if (!reuse_gram) {
      if (int st = launch_gram(p, Y, dt, G, RecordArgs{}, ranked, s)) return st;
    }
    {
      Timed t("routing_prep", s);
      // threads (= tokens) per workgroup: as many as fit 64 KB of LDS with their records, 64 at least
      int tpb = 256;
      while (tpb > 64 && (size_t)(p.rec_floats + 1) * tpb * sizeof(float) > 64 * 1024) tpb >>= 1;
      const size_t lds = (size_t)(p.rec_floats + 1) * tpb * sizeof(float);
      const bool staged = lds <= 64 * 1024;
      if (!staged) tpb = 256;
      const dim3 grid((unsigned)ceil_div(p.T, tpb));
      const bool vec = logits_vec(logits, p.E);
      unsigned long long* const clear = (unsigned long long*)unaffected;
#define MOEP_PREP_LAUNCH(EMAX, CAP)                                                                                 \
  do {                                                                                                              \
    if (staged)                                                                                                     \
      hipLaunchKernelGGL((prep_kernel<EMAX, CAP, true>), grid, dim3(tpb), lds, s, logits, G, rec, p.T, p.E, vec,    \
                         p.k, p.n_act, cap, p.rec_floats, clear);                                                   \
    else                                                                                                            \
      hipLaunchKernelGGL((prep_kernel<EMAX, CAP, false>), grid, dim3(tpb), 0, s, logits, G, rec, p.T, p.E, vec,     \
                         p.k, p.n_act, cap, p.rec_floats, clear);                                                   \
  } while (0)
#define MOEP_PREP_CAPS(EMAX)                                                                                        \
  switch (cap) {                                                                                                    \
    case 2: MOEP_PREP_LAUNCH(EMAX, 2); break;                                                                       \
    case 4: MOEP_PREP_LAUNCH(EMAX, 4); break;                                                                       \
    case 6: MOEP_PREP_LAUNCH(EMAX, 6); break;                                                                       \
    case 8: MOEP_PREP_LAUNCH(EMAX, 8); break;                                                                       \
    case 12: MOEP_PREP_LAUNCH(EMAX, 12); break;                                                                     \
    default: MOEP_PREP_LAUNCH(EMAX, 0); break;                                                                      \
  }
      if (p.E <= 8) { MOEP_PREP_CAPS(8) }
      else if (p.E <= 16) { MOEP_PREP_CAPS(16) }
      else { MOEP_PREP_CAPS(32) }
#undef MOEP_PREP_CAPS
#undef MOEP_PREP_LAUNCH
      MOEP_HIP(hipGetLastError());
    }
    if (int st = launch_scores(p, rec, partial, pcnt, ws, unaffected, s)) return st;
  }
  return launch_reduce_argmin(partial, p.fused_threads ? nullptr : pcnt, p.T > 0 ? p.n_tok_tiles : 0, p.n_sub, p.E, p.r, job.loss,
                              job.argmin, job.argmin_mask, unaffected, p.T > 0, s);
}

// Partial sums of one r that one workgroup reduces as fast as two launches follow each other, one of them over the whole chip.
// One / two, us: 70 subsets, 5500 tokens (12040 sums) 13.5 / -, 7000 16.1 / 10.2, 8192 18.2 / 10.0; 28 subsets, 16384 tokens (14336)
// 12.5 / 9.7; 120 subsets, 4001 tokens 13.4 / 11.2.
constexpr int64_t REDUCE_ONE_MAX = 12288;

// `cleared`: the counters are 0 already.  How a job is reduced depends on that job alone, so that an r gives the same bits by
// itself and among others; jobs that are reduced alike share the launches.
static int reduce_argmin(const ReduceSet& set, int E, bool cleared, hipStream_t s) {
  Timed t("loss_reduce_argmin", s);
  for (int subs : {0, 1, 32}) {                            // in one workgroup; by reduce_kernel<1>, <32>
    ReduceSet part = {};
    uint32_t blocks = 0;
    for (int i = 0; i < set.n; ++i) {
      ReduceJob j = set.job[i];
      const bool one = j.n_tiles * j.n_sub <= REDUCE_ONE_MAX && j.n_sub <= REDUCE_ONE_MAX;
      if (subs != (one ? 0 : j.n_sub >= 1024 ? 32 : 1)) continue;
      if (!j.partial_cnt) j.unaffected = nullptr;          // counted elsewhere
      if (one) {
        for (j.S = 1; j.S < (int)j.n_sub && j.S < 1024;) j.S <<= 1;
      } else {
        if (j.unaffected && !cleared) hipLaunchKernelGGL(zero_i64_kernel, dim3(1), dim3(1), 0, s, j.unaffected);
        j.first_block = blocks;
        blocks += (uint32_t)ceil_div(j.n_sub, subs);
      }
      part.job[part.n++] = j;
    }
    if (part.n == 0) continue;
    if (subs == 0) {
      hipLaunchKernelGGL(reduce_one_kernel, dim3(part.n), dim3(1024), 0, s, part, E);
    } else {
      if (subs == 32) hipLaunchKernelGGL(reduce_kernel<32>, dim3(blocks), dim3(256), 0, s, part);
      else hipLaunchKernelGGL(reduce_kernel<1>, dim3(blocks), dim3(256), 0, s, part);
      hipLaunchKernelGGL(argmin_kernel, dim3(part.n), dim3(1024), 0, s, part, E);
    }
    MOEP_HIP(hipGetLastError());
  }
  return MOEP_OK;
}

int launch_reduce_argmin(const float* partial, const uint32_t* pcnt, int64_t n_tiles, int64_t n_sub, int E, int r,
                         float* loss, int32_t* argmin, uint32_t* argmin_mask, int64_t* unaffected, bool cleared,
                         hipStream_t s) {
  ReduceSet set = {};
  set.n = 1;
  set.job[0] = {partial, pcnt, n_tiles, (uint32_t)n_sub, 0, 0, r, loss, (unsigned long long*)unaffected, argmin, argmin_mask};
  return reduce_argmin(set, E, cleared, s);
}

int launch_enumerate(const EnumJob* jobs, int n, const float* logits, const void* Y, moep_dtype dt, char* ws, size_t ws_bytes,
                     hipStream_t s, const RankedSource* ranked) {
  const EnumPlan* plans[RECORD_SETS];
  for (int i = 0; i < n; ++i) plans[i] = &jobs[i].plan;
  const EnumPlan& p0 = jobs[0].plan;
  RecordPlan at;
  if (!gram_writes_records(p0, Y, dt) ||
      !records_by_gram_pass(plans, n, ranked ? ranked->n_rank : 0, dt != MOEP_BF16, ws_bytes, &at)) {
    for (int i = 0; i < n; ++i)
      if (int st = launch_enumerate_from_gram(jobs[i], logits, Y, dt, ws, s, ranked, i > 0)) return st;
    return MOEP_OK;
  }
  RecordArgs recs = {};
  recs.logits = logits;
  recs.n = n;
  recs.k = p0.k;
  ReduceSet set = {};
  set.n = n;
  for (int i = 0; i < n; ++i) {
    const EnumJob& j = jobs[i];
    const EnumPlan& p = j.plan;
    recs.set[i] = {(float*)(ws + at.rec[i]), (unsigned long long*)j.unaffected, capacity_for(p.n_act), p.n_act, p.rec_floats};
    set.job[i] = {(const float*)(ws + at.partial[i]), p.fused_threads ? nullptr : (const uint32_t*)(ws + at.cnt[i]), p.n_tok_tiles,
                  (uint32_t)p.n_sub, 0, 0, p.r, j.loss, (unsigned long long*)j.unaffected, j.argmin, j.argmin_mask};
  }
  if (int st = launch_gram(p0, Y, dt, nullptr, recs, ranked, s)) return st;
  for (int i = 0; i < n; ++i)
    if (int st = launch_scores(jobs[i].plan, recs.set[i].rec, (float*)(ws + at.partial[i]), (uint32_t*)(ws + at.cnt[i]), ws,
                               jobs[i].unaffected, s)) return st;
  return reduce_argmin(set, p0.E, true, s);
}

int launch_subset_masks(int E, int r, int64_t n_sub, uint32_t* masks, hipStream_t s) {
  hipLaunchKernelGGL(masks_kernel, dim3((unsigned)ceil_div(n_sub, 256)), dim3(256), 0, s, E, r, (uint32_t)n_sub, masks);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
