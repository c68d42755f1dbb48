// Dynamic skipping, top-2 (Sec. 3.3; output per App. A.2): routing, dispatch and combine.
// The expert FFNs themselves are the grouped GEMMs (see gemm_bf16_packed.hip / gemm_few.hip / gemm_f32.hip).
//
//   route    per token: top-2 experts by logit among the kept experts (ties -> lower index), delta = l_e1 - l_e0 in fp32,
//            skip iff delta < theta = fp32(ln beta) (theta = -inf for beta = 0), weights
//            a0 = 1 / (1 + rho), a1 = rho / (1 + rho), rho = exp(delta); a0 = 1 when skipped.
//            Also counts, per block of 256 tokens, the rows each expert receives.
//   place    turns the counts into each (block, expert)'s first slot and each expert's segment end, and writes the map from
//            M tiles (256 or 192 rows, or 64) to (expert, first row) that the grouped bf16 GEMMs walk (entry [max_tiles] of the
//            expert list holds the number of tiles in use), for the 256-row GEMM the order in which they walk it, the slot -> token and
//            slot -> weight lists and the token -> slot positions.  Within an expert's segment the rows are in ascending
//            token order, so the result is reproducible.
//            (batches of up to dispatch_one_tokens, 256 to 1024, go through route and place in ONE workgroup, dispatch_one; beyond
//            65536 tokens a kernel of its own, scan, turns the counts into first slots)
//   combine  out[t] = slot_out[pos0] (+ slot_out[pos1] unless skipped); the down projection has
//            already multiplied each slot by its weight.  No atomics anywhere on this path.
//
// The *_topk kernels are the same pipeline for the generalised rule of the theory appendix: each
// token keeps the top-i* of its top-k experts, i* = min { i : sum_{m>i} w_m <= beta sum_{m<=k} w_m },
// decided in fp64 on the fp32 logits (tail sums accumulated from the smallest weight upwards), and
// the kept weights are renormalised over those i*.
#include <cmath>

#include "common.h"
#include "router_few.h"

namespace moep {
namespace {

constexpr int RB = 256;     // tokens per routing block
// Most routing blocks whose counts every workgroup of the place kernel adds up for itself (E 8: 8 KB of counts each).
constexpr int64_t PLACE_MAX_BLOCKS = 256;

struct Top2 { int e0, e1; float a0, a1; bool skip; };

// The top-2 rule on row t of the logits.
template <int EMAX>
__device__ __forceinline__ Top2 route_top2(const float* logits, int64_t t, int E, bool vec, uint32_t kept, float theta) {
  float v[EMAX];
  load_logits<EMAX>(logits, t, E, vec, v);
  const TopTwo t2 = top_two<EMAX>(v, E, kept);
  const float delta = t2.l1 - t2.l0;
  const bool skip = delta < theta;
  const float rho = expf(delta);
  return {t2.e0, t2.e1, skip ? 1.0f : 1.0f / (1.0f + rho), skip ? 0.0f : rho / (1.0f + rho), skip};
}

template <int EMAX>
__global__ __launch_bounds__(RB) void route_kernel(const float* __restrict__ logits, int64_t T,
                                                   int E, bool vec, uint32_t kept, float theta,
                                                   uint8_t* __restrict__ skip_mask, int32_t* __restrict__ top2,
                                                   float* __restrict__ tw, int32_t* __restrict__ counts) {
  __shared__ int cnt[32];
  if (threadIdx.x < 32) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * RB + threadIdx.x;
  if (t < T) {
    const Top2 r = route_top2<EMAX>(logits, t, E, vec, kept, theta);
    skip_mask[t] = r.skip ? 1 : 0;
    top2[2 * t] = r.e0;
    top2[2 * t + 1] = r.e1;
    tw[2 * t] = r.a0;
    tw[2 * t + 1] = r.a1;
    atomicAdd(&cnt[r.e0], 1);
    if (!r.skip) atomicAdd(&cnt[r.e1], 1);
  }
  __syncthreads();
  if ((int)threadIdx.x < E) counts[(int64_t)blockIdx.x * E + threadIdx.x] = cnt[threadIdx.x];
}

// The experts' segments and tiles from their row counts, by one wavefront: lane e < E holds expert e's count.  publish: to
// memory as well.
struct Segments { int32_t* seg_end; int32_t* tile_expert; int max_tiles, tile_rows; Shorten shorten; };
struct Layout { int begin[33], first_tile[33], rows_of_tile, most_rows; };         // in LDS; the first two [E + 1]
__device__ __forceinline__ void lay_out_segments(int lane, int E, int count, const Segments& s, Layout& out, bool publish) {
  const int c = lane < E ? count : 0;
  int tile_rows = s.tile_rows, most = c;
  if (s.shorten.n_up != 0) {                     // the 256-row GEMMs
    int tall = (c + GEMM_BM - 1) / GEMM_BM, shortened = (c + SHORT_TILE_ROWS - 1) / SHORT_TILE_ROWS;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      tall += __shfl_xor(tall, off, 64);
      shortened += __shfl_xor(shortened, off, 64);
      const int m = __shfl_xor(most, off, 64);
      most = m > most ? m : most;
    }
    if (shortened <= s.max_tiles && short_tiles_pay(s.shorten, tall, shortened)) tile_rows = SHORT_TILE_ROWS;
  }
  const int tiles = (c + tile_rows - 1) / tile_rows;
  int end = c, tile_end = tiles;                 // inclusive sums over the lanes
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int a = __shfl_up(end, off, 64), b = __shfl_up(tile_end, off, 64);
    end += lane >= off ? a : 0;
    tile_end += lane >= off ? b : 0;
  }
  if (lane <= E) {
    out.begin[lane] = end - c;
    out.first_tile[lane] = tile_end - tiles;
    if (publish) {
      s.seg_end[E + lane] = tile_end - tiles;
      if (lane < E) s.seg_end[lane] = end;
    }
  }
  if (lane == E) {
    if (publish) {
      s.tile_expert[s.max_tiles] = tile_end;     // number of tiles in use, read by the packing of x and by the few-rows GEMM
      s.seg_end[2 * E + 1] = tile_rows;
    }
    out.rows_of_tile = tile_rows;
    out.most_rows = most;
  }
}

// The expert whose tiles, n_tiles per M tile, tile q is one of: the last e with first_tile[e] n_tiles <= q (five look-ups;
// expert after expert it was one per expert, each waiting for the one before).
__device__ __forceinline__ int expert_of_tile(const Layout& l, int E, uint32_t n_tiles, uint32_t q) {
  int e = 0;
#pragma unroll
  for (int step = 16; step >= 1; step >>= 1)
    if (e + step < E && (uint32_t)l.first_tile[e + step] * n_tiles <= q) e += step;
  return e;
}

// The map of tiles, entries i0, i0 + step, ...
__device__ __forceinline__ void write_tile_map(const Layout& l, int E, const Segments& seg, int32_t* tile_row0, int64_t i0, int64_t step) {
  for (int64_t i = i0; i < seg.max_tiles; i += step) {
    const bool used = i < l.first_tile[E];
    const int e = expert_of_tile(l, E, 1, (uint32_t)i);
    seg.tile_expert[i] = used ? e : -1;
    tile_row0[i] = used ? l.begin[e] + ((int)i - l.first_tile[e]) * l.rows_of_tile : 0;
  }
}

// The order in which a grouped GEMM launch walks its tiles.  The launch gives every XCD a contiguous run of this
// list; within a run, 32 consecutive entries are in flight together and share operand panels through the XCD's L2.
// Entries are grouped per EXPERT: group_m consecutive M tiles of one expert, walked along N (all group_m tiles of
// one N tile, then the next N tile), so that the tiles in flight share the same few weight panels; an expert's last
// group may be smaller.  Entry = (M tile << 12) | N tile.  The width of the tiles is decided here, from the number of tiles the
// routing made, and noted in the header.  A thread takes tiles q0, q0 + step, ...
struct OrderArgs { uint32_t* order; int n_full, n_half, group_m, k; };     // order NULL: none is wanted
__device__ __forceinline__ void write_order(const Layout& l, int E, const OrderArgs& a, uint32_t q0, uint32_t step) {
  const int row_groups = gemm_row_groups(l.most_rows < l.rows_of_tile ? l.most_rows : l.rows_of_tile);
  const uint32_t m_tiles = (uint32_t)l.first_tile[E], tiles = m_tiles * (uint32_t)a.n_full;
  const bool half = half_width_pays(tiles);
  const uint32_t n_tiles = (uint32_t)(half ? a.n_half : a.n_full), most_m = (uint32_t)(half ? a.group_m / 2 : a.group_m);
  const uint32_t tail = (uint32_t)tail_tiles(tiles, a.n_full, a.n_half, a.k, row_groups), full = half ? 0u : tiles - tail;
  if (q0 == 0) {
    a.order[TILE_ORDER_HALF] = half ? m_tiles * n_tiles : 2 * tail;
    a.order[TILE_ORDER_FULL] = full;
    a.order[TILE_ORDER_ROW_GROUPS] = (uint32_t)row_groups;
  }
  for (uint32_t q = q0; q < m_tiles * n_tiles; q += step) {
    const int e = expert_of_tile(l, E, n_tiles, q);
    const uint32_t first = (uint32_t)l.first_tile[e], qe = q - first * n_tiles, c = (uint32_t)l.first_tile[e + 1] - first;
    const uint32_t g = qe / (most_m * n_tiles), first_m = g * most_m, gm = c - first_m < most_m ? c - first_m : most_m;
    const uint32_t in_group = qe - g * (most_m * n_tiles), tn = in_group / gm, row = (first + first_m + in_group - tn * gm) << 12;
    if (tail > 0 && q >= full) {                           // (an odd number of half tiles along N: the last one has no columns)
      a.order[TILE_ORDER_HEADER + 2 * q - full] = row | (2 * tn);
      a.order[TILE_ORDER_HEADER + 2 * q - full + 1] = row | (2 * tn + 1);
    } else {
      a.order[TILE_ORDER_HEADER + q] = row | tn;
    }
  }
}

// seg_end holds 2 E + 2 ints: the E segment ends, then the index of each expert's first tile (E + 1 entries,
// the last one being the number of tiles in use), then the rows per tile.  One workgroup: strands of consecutive routing blocks are summed per
// expert, and a scan over the strands gives each its base (one thread per expert over all blocks: the dispatch of 32768 tokens
// took 45 us with that, 18 so).
constexpr int SCAN_THREADS = 1024;
__global__ __launch_bounds__(SCAN_THREADS) void scan_kernel(int32_t* __restrict__ counts, int64_t n_blocks,
                                                   int E, Segments seg) {
  __shared__ int part[SCAN_THREADS];           // [strand][32 experts]
  __shared__ Layout lay;
  constexpr int STRANDS = SCAN_THREADS / 32;
  const int e = threadIdx.x & 31, strand = threadIdx.x >> 5;
  const int64_t per = (n_blocks + STRANDS - 1) / STRANDS;
  const int64_t b0 = strand * per < n_blocks ? strand * per : n_blocks;
  const int64_t b1 = b0 + per < n_blocks ? b0 + per : n_blocks;
  int sum = 0;
  if (e < E)
    for (int64_t b = b0; b < b1; ++b) sum += counts[b * E + e];
  part[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < STRANDS; off <<= 1) {    // inclusive sums over the strands
    const int v = strand >= off ? part[threadIdx.x - 32 * off] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  if (threadIdx.x < 64)
    lay_out_segments(threadIdx.x, E, part[(STRANDS - 1) * 32 + (threadIdx.x & 31)], seg, lay, true);
  __syncthreads();
  if (e < E) {
    int run = lay.begin[e] + part[threadIdx.x] - sum;
    for (int64_t b = b0; b < b1; ++b) {
      const int c = counts[b * E + e];
      counts[b * E + e] = run;
      run += c;
    }
  }
}

__device__ __forceinline__ uint32_t bf16_rne(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

template <bool BF16>
__global__ __launch_bounds__(256) void combine_kernel(const float4* __restrict__ slot_out,
                                                      const int32_t* __restrict__ pos, int64_t T,
                                                      int H4, void* __restrict__ out, bool singles_done) {
  const int64_t n = T * H4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t t = i / H4;
    const int c = (int)(i - t * H4);
    const int p0 = pos[2 * t], p1 = pos[2 * t + 1];
    if (singles_done && p1 < 0) continue;       // written by the down projection
    float4 v = slot_out[(int64_t)p0 * H4 + c];
    if (p1 >= 0) {
      const float4 u = slot_out[(int64_t)p1 * H4 + c];
      v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    if (BF16) {
      uint2 o;
      o.x = bf16_rne(v.x) | (bf16_rne(v.y) << 16);
      o.y = bf16_rne(v.z) | (bf16_rne(v.w) << 16);
      ((uint2*)out)[i] = o;
    } else {
      ((float4*)out)[i] = v;
    }
  }
}


// ---- generalised top-k skipping -----------------------------------------------------------
// The generalised rule on one row of logits: the top-K experts es, best first, the number istar that stays, and
// the renormalised weights of those (0 for the others).
template <int K, int EMAX>
__device__ __forceinline__ int route_topk(const float* logits, int64_t t, int E, bool vec, uint32_t kept, double beta,
                                          int (&es)[K], float (&w)[K]) {
  float l[EMAX];
  load_logits<EMAX>(logits, t, E, vec, l);
  uint32_t avail = kept;
  double ex[K];
  float l_first = 0.f;
#pragma unroll
  for (int m = 0; m < K; ++m) {            // m-th largest kept logit; strict >: lower index wins a tie
    int best = -1;
    float bv = 0.f;
#pragma unroll
    for (int e = 0; e < EMAX; ++e)
      if (((avail >> e) & 1u) && (best < 0 || l[e] > bv)) { best = e; bv = l[e]; }
    avail &= ~(1u << best);
    es[m] = best;
    if (m == 0) l_first = bv;
    ex[m] = exp((double)bv - (double)l_first);
  }
  double tail[K + 1];                      // tail[i] = sum_{m > i} w_m (m counted from 1)
  tail[K] = 0.0;
#pragma unroll
  for (int i = K - 1; i >= 0; --i) tail[i] = tail[i + 1] + ex[i];
  const double budget = beta * tail[0];
  int istar = K;
#pragma unroll
  for (int i = K - 1; i >= 1; --i)
    if (!(tail[i] > budget)) istar = i;    // ends at the smallest i that passes; tail[K] = 0 always passes
  // tails shrink with i, so "passes" is monotone and the smallest passing i is the answer
  double den = 0.0;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m < istar) den += ex[m];
#pragma unroll
  for (int m = 0; m < K; ++m) w[m] = m < istar ? (float)(ex[m] / den) : 0.0f;
  return istar;
}

template <int K, int EMAX>
__global__ __launch_bounds__(RB) void route_topk_kernel(const float* __restrict__ logits, int64_t T,
                                                        int E, bool vec, uint32_t kept, double beta,
                                                        int32_t* __restrict__ n_used,
                                                        int32_t* __restrict__ topk,
                                                        float* __restrict__ tw,
                                                        int32_t* __restrict__ counts) {
  __shared__ int cnt[32];
  if (threadIdx.x < 32) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * RB + threadIdx.x;
  if (t < T) {
    int es[K];
    float w[K];
    const int istar = route_topk<K, EMAX>(logits, t, E, vec, kept, beta, es, w);
    n_used[t] = istar;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      topk[t * K + m] = es[m];
      tw[t * K + m] = w[m];
      if (m < istar) atomicAdd(&cnt[es[m]], 1);
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < E) counts[(int64_t)blockIdx.x * E + threadIdx.x] = cnt[threadIdx.x];
}

// Workgroups 0 .. blocks of 256 tokens - 1 place their tokens' slots, the others write the tile orders.  scanned: counts
// holds first slots and the layout is in seg.seg_end; otherwise every workgroup adds up the counts of all blocks.
// TOP2: the top-2 rule with its skip mask; else the generalised rule with its counts.
template <int K, bool TOP2>
__global__ __launch_bounds__(RB) void place_kernel(const int32_t* __restrict__ experts, const float* __restrict__ tw,
                                                   const uint8_t* __restrict__ skip_mask, const int32_t* __restrict__ n_used,
                                                   const int32_t* __restrict__ counts, int n_blocks, bool scanned, int64_t T, int E,
                                                   int32_t* __restrict__ slot_token, float* __restrict__ slot_scale,
                                                   int32_t* __restrict__ slot_dest, int32_t* __restrict__ pos,
                                                   int32_t* __restrict__ tile_row0, Segments seg, OrderArgs up, OrderArgs down) {
  constexpr int STRANDS = RB / 32;
  __shared__ int total[RB], before[RB];        // [strand][32 experts]
  __shared__ int wave_cnt[RB / 64][32];
  __shared__ Layout lay;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int block = blockIdx.x;
  const int e32 = tid & 31, strand = tid >> 5;
  if (scanned) {
    if (tid <= E) {
      lay.begin[tid] = tid ? seg.seg_end[tid - 1] : 0;
      lay.first_tile[tid] = seg.seg_end[E + tid];
    }
    if (tid == 0) {
      int most = 0;
      for (int e = 0, last = 0; e < E; ++e) {
        const int end = seg.seg_end[e];
        most = end - last > most ? end - last : most;
        last = end;
      }
      lay.most_rows = most;
      lay.rows_of_tile = seg.seg_end[2 * E + 1];
    }
    if (tid < E && block < n_blocks) before[tid] = counts[(int64_t)block * E + tid];
    __syncthreads();
  } else {
    int all = 0, mine = 0;
    if (e32 < E)
#pragma unroll 4
      for (int b = strand; b < n_blocks; b += STRANDS) {
        const int c = counts[b * E + e32];
        all += c;
        mine += b < block ? c : 0;
      }
    total[tid] = all;
    before[tid] = mine;
    __syncthreads();
    if (tid < 64) {
      all = mine = 0;
#pragma unroll
      for (int s = 0; s < STRANDS; ++s) {
        all += total[s * 32 + e32];
        mine += before[s * 32 + e32];
      }
      lay_out_segments(lane, E, all, seg, lay, block == 0);
      if (lane < E) before[lane] = lay.begin[lane] + mine;           // (lane's own entry; all sums of the wavefront are done)
    }
    __syncthreads();
  }
  write_tile_map(lay, E, seg, tile_row0, (int64_t)block * RB + tid, (int64_t)gridDim.x * RB);
  if (block >= n_blocks) {
    const uint32_t q = (uint32_t)(block - n_blocks) * RB + tid, step = (gridDim.x - n_blocks) * RB;
    write_order(lay, E, up, q, step);
    write_order(lay, E, down, q, step);
    return;
  }
  const int64_t t = (int64_t)block * RB + tid;
  const bool live = t < T;
  const int nu = !live ? 0 : TOP2 ? (skip_mask[t] ? 1 : 2) : n_used[t];
  int es[K], rank[K];
#pragma unroll
  for (int m = 0; m < K; ++m) { es[m] = m < nu ? experts[t * K + m] : -1; rank[m] = 0; }
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int e = 0; e < E; ++e) {             // a token routes to an expert at most once
    bool has = false;
#pragma unroll
    for (int m = 0; m < K; ++m) has |= es[m] == e;
    const unsigned long long b = __ballot(has);
    const int ahead = __popcll(b & below);
#pragma unroll
    for (int m = 0; m < K; ++m)
      if (es[m] == e) rank[m] = ahead;
    if (lane == 0) wave_cnt[wave][e] = __popcll(b);
  }
  __syncthreads();
  if (!live) return;
#pragma unroll
  for (int m = 0; m < K; ++m) {
    int p = -1;
    if (es[m] >= 0) {
      p = before[es[m]] + rank[m];
      for (int w = 0; w < wave; ++w) p += wave_cnt[w][es[m]];
      slot_token[p] = (int32_t)t;
      slot_scale[p] = tw[t * K + m];
      slot_dest[p] = nu == 1 ? (int32_t)t : -1;     // a token's only slot (weight 1) is the token's output
    }
    pos[t * K + m] = p;
  }
}

template <bool BF16>
__global__ __launch_bounds__(256) void combine_topk_kernel(const float4* __restrict__ slot_out,
                                                           const int32_t* __restrict__ pos, int64_t T,
                                                           int H4, int K, void* __restrict__ out, bool singles_done) {
  const int64_t n = T * H4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t t = i / H4;
    const int c = (int)(i - t * H4);
    if (singles_done && (K == 1 || pos[t * K + 1] < 0)) continue;     // written by the down projection
    float4 v = slot_out[(int64_t)pos[t * K] * H4 + c];     // the best expert is always kept
    for (int m = 1; m < K; ++m) {
      const int p = pos[t * K + m];
      if (p < 0) break;                                   // kept experts are a prefix of the top-k
      const float4 u = slot_out[(int64_t)p * H4 + c];
      v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    if (BF16) {
      uint2 o;
      o.x = bf16_rne(v.x) | (bf16_rne(v.y) << 16);
      o.y = bf16_rne(v.z) | (bf16_rne(v.w) << 16);
      ((uint2*)out)[i] = o;
    } else {
      ((float4*)out)[i] = v;
    }
  }
}

// ---- the whole dispatch in one workgroup ----------------------------------------------------
// route and place for a batch that fits one workgroup (a thread per token): two launches, all of it latency, become one.
// Same outputs as the two, entry for entry.  tw is not written: the weights go straight to the slots.
struct Dispatch {
  const float* logits; int T, E; bool vec; uint32_t kept; float theta; double beta;
  uint8_t* skip_mask; int32_t* n_used; int32_t* experts; int32_t* slot_token; float* slot_scale; int32_t* slot_dest; int32_t* pos;
  int32_t* tile_row0; Segments seg; OrderArgs up, down;
};
template <int K, bool TOP2, int EMAX>
__device__ __forceinline__ void dispatch_one(const Dispatch& d) {
  const float* const logits = d.logits;                   // (may have been written by this workgroup)
  const int T = d.T, E = d.E;
  const bool vec = d.vec;
  const uint32_t kept = d.kept;
  const float theta = d.theta;
  const double beta = d.beta;
  uint8_t* __restrict__ const skip_mask = d.skip_mask;
  int32_t* __restrict__ const n_used = d.n_used;
  int32_t* __restrict__ const experts = d.experts;
  int32_t* __restrict__ const slot_token = d.slot_token;
  float* __restrict__ const slot_scale = d.slot_scale;
  int32_t* __restrict__ const slot_dest = d.slot_dest;
  int32_t* __restrict__ const pos = d.pos;
  int32_t* __restrict__ const tile_row0 = d.tile_row0;
  const Segments& seg = d.seg;
  const OrderArgs &up = d.up, &down = d.down;
  constexpr int WAVES = DISPATCH_ONE_MAX / 64;
  __shared__ int wave_base[WAVES][32];     // counts, then first slots, of (wavefront, expert)
  __shared__ Layout lay;
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const bool live = t < T;
  int es[K], rank[K], used = 0;
  float w[K];
#pragma unroll
  for (int m = 0; m < K; ++m) { es[m] = -1; rank[m] = 0; w[m] = 0.f; }
  if (live) {
    if constexpr (TOP2) {
      const Top2 r = route_top2<EMAX>(logits, t, E, vec, kept, theta);
      es[0] = r.e0; w[0] = r.a0;
      es[1] = r.e1; w[1] = r.a1;
      used = r.skip ? 1 : 2;
      skip_mask[t] = r.skip ? 1 : 0;
    } else {
      used = route_topk<K, EMAX>(logits, t, E, vec, kept, beta, es, w);
      n_used[t] = used;
    }
#pragma unroll
    for (int m = 0; m < K; ++m) {
      experts[t * K + m] = es[m];
      if (m >= used) es[m] = -1;
    }
  }
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int e = 0; e < E; ++e) {             // a token routes to an expert at most once
    bool has = false;
#pragma unroll
    for (int m = 0; m < K; ++m) has |= es[m] == e;
    const unsigned long long b = __ballot(has);
    const int before = __popcll(b & below);
#pragma unroll
    for (int m = 0; m < K; ++m)
      if (es[m] == e) rank[m] = before;
    if (lane == 0) wave_base[wave][e] = __popcll(b);
  }
  __syncthreads();
  const int waves = blockDim.x >> 6;
  if (wave == 0) {
    int run = 0;                            // slots before (wavefront, expert t) within the expert's segment, then its rows
    if (t < E)
      for (int v = 0; v < waves; ++v) {
        const int c = wave_base[v][t];
        wave_base[v][t] = run;
        run += c;
      }
    lay_out_segments(t, E, run, seg, lay, true);
  }
  __syncthreads();
  // the map of tiles, an expert's by its thread (with a look-up per tile, as in the place kernel, this launch takes 0.2 to 0.5 us more)
  if (t < E)
    for (int i = lay.first_tile[t]; i < lay.first_tile[t + 1]; ++i) {
      seg.tile_expert[i] = t;
      tile_row0[i] = lay.begin[t] + (i - lay.first_tile[t]) * lay.rows_of_tile;
    }
  for (int i = lay.first_tile[E] + t; i < seg.max_tiles; i += blockDim.x) {
    seg.tile_expert[i] = -1;
    tile_row0[i] = 0;
  }
  if (up.order) {
    write_order(lay, E, up, t, blockDim.x);
    write_order(lay, E, down, t, blockDim.x);
  }
  if (!live) return;
#pragma unroll
  for (int m = 0; m < K; ++m) {
    int p = -1;
    if (m < used) {
      p = lay.begin[es[m]] + wave_base[wave][es[m]] + rank[m];
      slot_token[p] = t;
      slot_scale[p] = w[m];
      slot_dest[p] = used == 1 ? t : -1;    // a token's only slot (weight 1) is the token's output
    }
    pos[t * K + m] = p;
  }
}

template <int K, bool TOP2, int EMAX>
__global__ __launch_bounds__(DISPATCH_ONE_MAX) void dispatch_one_kernel(Dispatch d) { dispatch_one<K, TOP2, EMAX>(d); }

// The router and the dispatch of up to 16 tokens in one launch: each is some 4 us of latency, on the GPU and in the host's queue.
// E 8, H 128, F 256, a call: 1 token 31.3 -> 26.9 us, 16 tokens 31.0 -> 27.0; one token of the Mixtral shape, both launches 8.1 ->
// 7.5, the call 72.0 -> 71.3.
constexpr int ROUTE_DISPATCH_MAX = 16, ROUTE_DISPATCH_SLOTS = 4;
template <int K, bool TOP2, int EMAX>
__global__ __launch_bounds__(512) void route_dispatch_kernel(const uint4* __restrict__ x, const uint4* __restrict__ Wgate, int H,
                                                             float* logits, Dispatch d) {
  if (d.E > 16) router_few<false, true, 8>(x, Wgate, logits, d.T, d.E, H, nullptr);
  else router_few<false, false, 8>(x, Wgate, logits, d.T, d.E, H, nullptr);
  __syncthreads();
  dispatch_one<K, TOP2, EMAX>(d);
}

}  // namespace

int plan_skip(int64_t T, int E, int H, int F, moep_dtype dt, int ks, int kept_experts, SkipPlan* p, bool with_slot_out) {
  if ((int64_t)ks * T >= ((int64_t)1 << 31)) return fail(MOEP_EUNSUPPORTED, "moe_forward_skip: T too large");
  p->T = T; p->E = E; p->H = H; p->F = F; p->ks = ks; p->kept_experts = kept_experts;
  p->max_slots = (int64_t)ks * T;
  p->few = dt == MOEP_BF16 && few_rows(T, ks, kept_experts, 3.0 * H * F * 2);
  p->tile_rows = p->few ? FEW_ROWS : GEMM_BM;
  p->max_tiles = ceil_div((int64_t)ks * T, p->tile_rows) + E;
  const int64_t map_tiles = ceil_div((int64_t)ks * T, dt == MOEP_BF16 ? FEW_ROWS : GEMM_BM) + E;   // either path's map fits
  const int64_t n_blocks = ceil_div(T, RB);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
  p->off_logits = take((size_t)T * E * 4);
  p->off_slot_token = take((size_t)p->max_slots * 4);
  p->off_slot_scale = take((size_t)p->max_slots * 4);
  p->off_slot_dest = take((size_t)p->max_slots * 4);
  p->off_pos = take((size_t)T * ks * 4 * 3);           // pos, experts, weights: [T,ks] each
  p->off_counts = take((size_t)n_blocks * E * 4);
  p->off_seg_end = take((size_t)(2 * E + 2) * 4);          // segment ends, then each expert's first tile, then rows per tile
  p->off_tile_expert = take((size_t)(map_tiles + 1) * 4);   // + the count of tiles in use
  p->off_tile_row0 = take((size_t)map_tiles * 4);
  p->packed = dt == MOEP_BF16;
  p->off_order_up = p->off_order_down = 0;
  if (dt == MOEP_BF16) {
    const int64_t gemm_tiles = ceil_div((int64_t)ks * T, GEMM_BM) + E;
    const int64_t n_up = ceil_div(F, gemm_tile_columns(true, true)), n_down = ceil_div(H, gemm_tile_columns(false, true));
    if (n_up > 4096 || n_down > 4096 || gemm_tiles >= (1 << 20))
      return fail(MOEP_EUNSUPPORTED, "moe_forward_skip: too many tiles for the tile order tables");
    p->off_order_up = take((size_t)(TILE_ORDER_HEADER + gemm_tiles * n_up) * 4);
    p->off_order_down = take((size_t)(TILE_ORDER_HEADER + gemm_tiles * n_down) * 4);
    // packed-operand GEMMs: h and the gathered x hold one 256-row block per tile; room for a packed copy of every
    // expert's weights, which calls with many rows per expert on row-major weights make
    p->off_h = take(packed_a_bytes(gemm_tiles * GEMM_BM, F));
    p->off_xp = take(packed_a_bytes(gemm_tiles * GEMM_BM, H));
    p->off_w13 = take((size_t)E * packed_b_bytes(F, H, true));
    p->off_w2 = take((size_t)E * packed_b_bytes(H, F, false));
  } else {
    p->off_h = take((size_t)p->max_slots * F * dtype_size(dt));
    p->off_xp = p->off_w13 = p->off_w2 = 0;
  }
  p->off_slot_out = take(with_slot_out ? (size_t)p->max_slots * H * 4 : 0);
  p->total = off > 0 ? off : 256;
  return MOEP_OK;
}

static Segments segments(const SkipPlan& p, char* ws) {
  Segments s = {(int32_t*)(ws + p.off_seg_end), (int32_t*)(ws + p.off_tile_expert), (int)p.max_tiles, p.tile_rows, {}};
  if (p.packed && !p.few) s.shorten = {(int)ceil_div(p.F, GEMM_BN_SWIGLU), (int)ceil_div(p.H, GEMM_BN_STORE), p.H, p.F};
  return s;
}

// Tile orders of the two grouped projections (bf16 path), and how many tiles of full width there can be.
struct Orders { OrderArgs up = {}, down = {}; int64_t entries = 0; };
static Orders orders(const SkipPlan& p, char* ws) {
  Orders o;
  if (!p.packed || p.few) return o;
  o.up = {(uint32_t*)(ws + p.off_order_up), (int)ceil_div(p.F, gemm_tile_columns(true, false)),
          (int)ceil_div(p.F, gemm_tile_columns(true, true)), GEMM_GROUP_M_SWIGLU, p.H};
  o.down = {(uint32_t*)(ws + p.off_order_down), (int)ceil_div(p.H, gemm_tile_columns(false, false)),
            (int)ceil_div(p.H, gemm_tile_columns(false, true)), GEMM_GROUP_M_STORE, p.F};
  o.entries = p.max_tiles * (o.up.n_full + o.down.n_full);
  return o;
}
static bool dispatch_in_one(const SkipPlan& p, const Orders& o) {
  return p.T <= dispatch_one_tokens(p.E, p.ks) && o.entries <= DISPATCH_ONE_ORDER_MAX;
}
// Its threads: one per token, and more of them where there are many tiles to put in order.
static unsigned dispatch_one_threads(const SkipPlan& p, const Orders& o) {
  const int64_t wanted = ceil_div(p.T, 64), tiles = ceil_div(o.entries, 2 * 64), most = DISPATCH_ONE_MAX / 64;
  return (unsigned)(64 * (wanted > tiles ? wanted : tiles < most ? tiles : most));
}

template <int K, bool TOP2>
static void launch_place(const SkipPlan& p, const Orders& o, const int32_t* experts, const float* tw, const uint8_t* skip_mask,
                         const int32_t* n_used, int32_t* pos, char* ws, hipStream_t s) {
  int32_t* counts = (int32_t*)(ws + p.off_counts);
  const int64_t n_blocks = ceil_div(p.T, RB);
  const bool scan = n_blocks > PLACE_MAX_BLOCKS;
  if (scan)
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(SCAN_THREADS), 0, s, counts, n_blocks, p.E, segments(p, ws));
  const int64_t order_blocks = ceil_div(o.entries, 2 * RB);
  hipLaunchKernelGGL((place_kernel<K, TOP2>), dim3((unsigned)(n_blocks + order_blocks)), dim3(RB), 0, s, experts, tw, skip_mask,
                     n_used, counts, (int)n_blocks, scan, p.T, p.E, (int32_t*)(ws + p.off_slot_token),
                     (float*)(ws + p.off_slot_scale), (int32_t*)(ws + p.off_slot_dest), pos, (int32_t*)(ws + p.off_tile_row0),
                     segments(p, ws), o.up, o.down);
}

bool routing_computes_logits(const SkipPlan& p, const void* x, const void* Wgate) {
  return p.packed && p.few && p.T <= ROUTE_DISPATCH_MAX && p.ks <= ROUTE_DISPATCH_SLOTS && mfma_router_applies(p.E, p.H) &&
         (((uintptr_t)x | (uintptr_t)Wgate) & 15) == 0 && dispatch_in_one(p, {});
}

int launch_skip_routing(const SkipPlan& p, const float* logits, uint32_t kept_mask, float beta, uint8_t* skip_mask,
                        int32_t* top2_out, char* ws, hipStream_t s, const void* x, const void* Wgate) {
  const int64_t T = p.T;
  int32_t* pos = (int32_t*)(ws + p.off_pos);
  int32_t* top2 = top2_out ? top2_out : pos + 2 * T;
  float* tw = (float*)(pos + 4 * T);
  int32_t* counts = (int32_t*)(ws + p.off_counts);
  const int64_t n_blocks = ceil_div(T, RB);
  const float theta = beta > 0.0f ? (float)std::log((double)beta) : -INFINITY;
  Timed t("skip_route_dispatch", s);
  const bool vec = logits_vec(logits, p.E);
  const Orders o = orders(p, ws);
  if (dispatch_in_one(p, o)) {
    const Dispatch d = {logits, (int)T, p.E, vec, kept_mask, theta, 0.0, skip_mask, nullptr, top2, (int32_t*)(ws + p.off_slot_token),
                        (float*)(ws + p.off_slot_scale), (int32_t*)(ws + p.off_slot_dest), pos, (int32_t*)(ws + p.off_tile_row0),
                        segments(p, ws), o.up, o.down};
#define MOEP_ONE(EMAX)                                                                                                    \
  do {                                                                                                                    \
    if (x)                                                                                                                \
      hipLaunchKernelGGL((route_dispatch_kernel<2, true, EMAX>), dim3(1), dim3(512), 0, s, (const uint4*)x,               \
                         (const uint4*)Wgate, p.H, (float*)logits, d);                                                    \
    else                                                                                                                  \
      hipLaunchKernelGGL((dispatch_one_kernel<2, true, EMAX>), dim3(1), dim3(dispatch_one_threads(p, o)), 0, s, d);       \
  } while (0)
    if (p.E <= 8) MOEP_ONE(8);
    else if (p.E <= 16) MOEP_ONE(16);
    else MOEP_ONE(32);
#undef MOEP_ONE
    MOEP_HIP(hipGetLastError());
    return MOEP_OK;
  }
#define MOEP_ROUTE(EMAX)                                                                                                \
  hipLaunchKernelGGL(route_kernel<EMAX>, dim3((unsigned)n_blocks), dim3(RB), 0, s, logits, T, p.E, vec, kept_mask, theta, \
                     skip_mask, top2, tw, counts)
  if (p.E <= 8) MOEP_ROUTE(8);
  else if (p.E <= 16) MOEP_ROUTE(16);
  else MOEP_ROUTE(32);
#undef MOEP_ROUTE
  launch_place<2, true>(p, o, top2, tw, skip_mask, nullptr, pos, ws, s);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

int launch_skip_combine(const SkipPlan& p, moep_dtype dt, const uint8_t* skip_mask, void* out,
                        char* ws, hipStream_t s, bool singles_done) {
  (void)skip_mask;
  const int H4 = p.H / 4;
  const int64_t n = p.T * H4;
  const unsigned blocks = (unsigned)(ceil_div(n, 256) < 65536 ? ceil_div(n, 256) : 65536);
  Timed t("skip_combine", s);
  if (dt == MOEP_BF16)
    hipLaunchKernelGGL(combine_kernel<true>, dim3(blocks), dim3(256), 0, s,
                       (const float4*)(ws + p.off_slot_out), (const int32_t*)(ws + p.off_pos), p.T, H4, out, singles_done);
  else
    hipLaunchKernelGGL(combine_kernel<false>, dim3(blocks), dim3(256), 0, s,
                       (const float4*)(ws + p.off_slot_out), (const int32_t*)(ws + p.off_pos), p.T, H4, out, singles_done);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}


int launch_skip_topk_routing(const SkipPlan& p, const float* logits, uint32_t kept_mask, float beta,
                             int32_t* n_used, int32_t* topk_out, char* ws, hipStream_t s, int32_t* pos_out, const void* x,
                             const void* Wgate) {
  const int64_t T = p.T;
  const int K = p.ks;
  int32_t* ws_pos = (int32_t*)(ws + p.off_pos);
  int32_t* pos = pos_out ? pos_out : ws_pos;
  int32_t* topk = topk_out ? topk_out : ws_pos + (int64_t)K * T;
  float* tw = (float*)(ws_pos + 2 * (int64_t)K * T);
  int32_t* counts = (int32_t*)(ws + p.off_counts);
  const int64_t n_blocks = ceil_div(T, RB);
  int32_t* slot_token = (int32_t*)(ws + p.off_slot_token);
  float* slot_scale = (float*)(ws + p.off_slot_scale);
  int32_t* slot_dest = (int32_t*)(ws + p.off_slot_dest);
  Timed t("skip_route_dispatch", s);
  const bool vec = logits_vec(logits, p.E);
  const Orders o = orders(p, ws);
  if (dispatch_in_one(p, o)) {
    const Dispatch d = {logits, (int)T, p.E, vec, kept_mask, 0.0f, (double)beta, nullptr, n_used, topk, slot_token, slot_scale,
                        slot_dest, pos, (int32_t*)(ws + p.off_tile_row0), segments(p, ws), o.up, o.down};
    if (x) {
#define MOEP_ROUTED_CASE(KK)                                                                                              \
  case KK:                                                                                                                \
    if (p.E <= 16)                                                                                                        \
      hipLaunchKernelGGL((route_dispatch_kernel<KK, false, 16>), dim3(1), dim3(512), 0, s, (const uint4*)x,               \
                         (const uint4*)Wgate, p.H, (float*)logits, d);                                                    \
    else                                                                                                                  \
      hipLaunchKernelGGL((route_dispatch_kernel<KK, false, 32>), dim3(1), dim3(512), 0, s, (const uint4*)x,               \
                         (const uint4*)Wgate, p.H, (float*)logits, d);                                                    \
    break;
      switch (K) {
        MOEP_ROUTED_CASE(1) MOEP_ROUTED_CASE(2) MOEP_ROUTED_CASE(3) MOEP_ROUTED_CASE(4)
        default: return fail(MOEP_EUNSUPPORTED, "routing with the router: k=%d (1..%d)", K, ROUTE_DISPATCH_SLOTS);
      }
#undef MOEP_ROUTED_CASE
      MOEP_HIP(hipGetLastError());
      return MOEP_OK;
    }
#define MOEP_ONE(KK, EMAX)                                                                                             \
  hipLaunchKernelGGL((dispatch_one_kernel<KK, false, EMAX>), dim3(1), dim3(dispatch_one_threads(p, o)), 0, s, d)
#define MOEP_ONE_CASE(KK)                                                                                              \
  case KK:                                                                                                             \
    if (p.E <= 16) MOEP_ONE(KK, 16);                                                                                   \
    else MOEP_ONE(KK, 32);                                                                                             \
    break;
    switch (K) {
      MOEP_ONE_CASE(1) MOEP_ONE_CASE(2) MOEP_ONE_CASE(3) MOEP_ONE_CASE(4)
      MOEP_ONE_CASE(5) MOEP_ONE_CASE(6) MOEP_ONE_CASE(7) MOEP_ONE_CASE(8)
      MOEP_ONE_CASE(9) MOEP_ONE_CASE(10) MOEP_ONE_CASE(11) MOEP_ONE_CASE(12)
      MOEP_ONE_CASE(13) MOEP_ONE_CASE(14) MOEP_ONE_CASE(15) MOEP_ONE_CASE(16)
      default: return fail(MOEP_EUNSUPPORTED, "top-k routing: k=%d (1..16)", K);
    }
#undef MOEP_ONE_CASE
#undef MOEP_ONE
    MOEP_HIP(hipGetLastError());
    return MOEP_OK;
  }
#define MOEP_ROUTE(KK, EMAX)                                                                                           \
  hipLaunchKernelGGL((route_topk_kernel<KK, EMAX>), dim3((unsigned)n_blocks), dim3(RB), 0, s, logits, T, p.E, vec,       \
                     kept_mask, (double)beta, n_used, topk, tw, counts)
#define MOEP_ROUTE_CASE(KK)                                                                                            \
  case KK:                                                                                                             \
    if (p.E <= 16) MOEP_ROUTE(KK, 16);                                                                                 \
    else MOEP_ROUTE(KK, 32);                                                                                           \
    break;
  switch (K) {
    MOEP_ROUTE_CASE(1) MOEP_ROUTE_CASE(2) MOEP_ROUTE_CASE(3) MOEP_ROUTE_CASE(4)
    MOEP_ROUTE_CASE(5) MOEP_ROUTE_CASE(6) MOEP_ROUTE_CASE(7) MOEP_ROUTE_CASE(8)
    MOEP_ROUTE_CASE(9) MOEP_ROUTE_CASE(10) MOEP_ROUTE_CASE(11) MOEP_ROUTE_CASE(12)
    MOEP_ROUTE_CASE(13) MOEP_ROUTE_CASE(14) MOEP_ROUTE_CASE(15) MOEP_ROUTE_CASE(16)
    default: return fail(MOEP_EUNSUPPORTED, "top-k routing: k=%d (1..16)", K);
  }
#undef MOEP_ROUTE_CASE
#undef MOEP_ROUTE
#define MOEP_SCATTER_CASE(KK)                                                                  \
  case KK: launch_place<KK, false>(p, o, topk, tw, nullptr, n_used, pos, ws, s); break;
  switch (K) {
    MOEP_SCATTER_CASE(1) MOEP_SCATTER_CASE(2) MOEP_SCATTER_CASE(3) MOEP_SCATTER_CASE(4)
    MOEP_SCATTER_CASE(5) MOEP_SCATTER_CASE(6) MOEP_SCATTER_CASE(7) MOEP_SCATTER_CASE(8)
    MOEP_SCATTER_CASE(9) MOEP_SCATTER_CASE(10) MOEP_SCATTER_CASE(11) MOEP_SCATTER_CASE(12)
    MOEP_SCATTER_CASE(13) MOEP_SCATTER_CASE(14) MOEP_SCATTER_CASE(15) MOEP_SCATTER_CASE(16)
  }
#undef MOEP_SCATTER_CASE
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

int launch_skip_topk_combine(const SkipPlan& p, moep_dtype dt, void* out, char* ws, hipStream_t s, bool singles_done) {
  const int H4 = p.H / 4;
  const int64_t n = p.T * H4;
  const unsigned blocks = (unsigned)(ceil_div(n, 256) < 65536 ? ceil_div(n, 256) : 65536);
  Timed t("skip_combine", s);
  if (dt == MOEP_BF16)
    hipLaunchKernelGGL(combine_topk_kernel<true>, dim3(blocks), dim3(256), 0, s,
                       (const float4*)(ws + p.off_slot_out), (const int32_t*)(ws + p.off_pos), p.T, H4, p.ks, out, singles_done);
  else
    hipLaunchKernelGGL(combine_topk_kernel<false>, dim3(blocks), dim3(256), 0, s,
                       (const float4*)(ws + p.off_slot_out), (const int32_t*)(ws + p.off_pos), p.T, H4, p.ks, out, singles_done);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
