// bf16 expert GEMMs for FEW rows per expert (token generation, small batches): C = epilogue(A B^T), fp32 accumulate.
//
// With a few dozen rows per expert the work is a read of the weights: 2 flop per weight byte and row, so the launch
// is bound by the memory from one row to about a hundred.  The 256-row tiles of gemm_bf16_packed.hip cannot reach that
// bound: one token leaves most compute units without a tile (the down projection of 4096 x 14336 has 16 tiles per
// expert, each a serial walk over 448 slices: 251 us for one token), and the padding rows are multiplied all the same.
//
// Here a weight element goes from memory through a wavefront's own LDS ring into the register of the one wavefront that
// multiplies it; nothing is shared and there is no barrier.  A wavefront takes 32 output columns (gate/up: 32 gate and the
// 32 up rows of the same columns) x up to 64 rows and walks all of K.  What keeps the memory busy is the bytes in flight: with
// 16 KB rings eight wavefronts fit a compute unit, and a launch of no more than four per compute unit takes rings of 40 KB
// instead (DEEP_RING), 12 to 36 KB of weights in flight for each.
// Rows of A (x through a token list, or h) are read as MFMA fragments from L1/L2: a few hundred KB.
//
// Weights come either as the caller stores them (row-major [N, K]) or in the blocked layout of moe_pack_weights; the same
// 16-row fragments, the same slices in the same order, so both give the same bits.  Every load is 1 KB straight into LDS:
// packed, a fragment's consecutive bytes; row-major, whole 128-byte lines of 8 rows.  (Fragment-shaped loads into registers
// ask for 64 bytes of 16 rows: row-major weights then came at 4.3 TB/s instead of 5.4; and from 64 rows on, the registers
// that the ring saves are worth 10 % on packed weights too.)
// Measured, skipping forward of the Mixtral shape (E 8, H 4096, F 14336) against the 256-row tiles: packed weights, one
// token 361 -> 75 us, 16 tokens (all 2.8 GB of weights) 732 -> 452 us = 6.2 TB/s, 128 tokens 750 -> 536 us; row-major
// weights, which needed a packing pass over all of them per call: 1510 -> 88 us, 1880 -> 500 us, 1880 -> 580 us.
// The products are summed in the order of gemm_packed_kernel (one v_mfma_f32_16x16x32_bf16 per slice, slices ascending),
// bit for bit, so that a token's outputs do not depend on the batch it comes in.  (Two to eight wavefronts sharing the
// columns, K split between them, fill the chip as well, but sum in an order that follows the size of the batch; one token
// took 79 us that way.)
#include <type_traits>

#include "common.h"

namespace moep {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int SLICE = 256 * 64;     // bytes of one packed block (256 rows x 32 k), see gemm_bf16_packed.hip
constexpr int RING = 16384, DEEP_RING = 40960;   // LDS of a wavefront's load ring
constexpr int DEEP_WAVES = 4;                    // wavefronts per compute unit up to which the deep ring is taken (they fit)
// Wavefronts of a workgroup.  Four with the small ring: they read neighbouring column groups in step (16 tokens, packed: the
// gate/up launch 290 us, 316 with workgroups of one).  One with the deep ring, so that few of them spread over the chip.
constexpr int waves_of(int ring) { return ring == DEEP_RING ? 1 : 4; }

struct FewArgs {
  const char* W0; const char* W1;     // row-major: W0 [N,K] (gate), W1 (up); packed: W0 = blocked copy
  int64_t w_expert_bytes;
  const char* X; int64_t x_row_bytes; // rows of A
  const int32_t* row_of;              // grouped gate/up: row r of the launch is row row_of[r] of X; NULL: r itself
  int64_t x_expert_rows;              // dense: rows between consecutive experts in X (0: shared)
  void* C; int64_t ldc;               // elements
  int64_t c_expert_rows;              // dense
  int N, nsl;                         // output columns; K / 32
  bool stream;                        // non-temporal weight loads
  // grouped: tile t = rows tile_row0[t] .. seg_end[tile_expert[t]] - 1, at most FEW_ROWS of them
  const int32_t* tile_expert; const int32_t* tile_row0; const int32_t* seg_end; const int32_t* tiles_in_use;
  // dense: tile t = rows (t % row_tiles) * FEW_ROWS .. of expert t / row_tiles
  int row_tiles; int64_t rows;
  const float* row_scale;
  const int32_t* row_dest; uint16_t* direct_out;
};

// Waits until no more than N vector-memory loads are in flight; they complete in issue order.  The compiler does not count
// direct loads into LDS against the reads of it, so N has to be what is issued after the loads that are waited for, exactly.
template <int N>
__device__ __forceinline__ void wait_until_flying() {
  static_assert(N < 64, "more loads in flight than the counter holds");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_sched_barrier(0);
}

// One tile, M groups of 16 rows (M >= the groups in use; rows beyond row_end repeat the last one and are not stored).
template <int EPI, bool PACKED, int M, bool STREAM, int RING_BYTES>
__device__ __forceinline__ void few_tile(const FewArgs& p, int n0, int expert, int64_t row0, int64_t row_end, char* ring) {
  constexpr int NF = EPI == EPI_SWIGLU ? 4 : 2;      // weight fragments of 16 rows: (gate, up) x 2 or 2
  constexpr int LOADS = 2 * NF + 2 * M;              // of a pair of slices
  // AHEAD: with few wavefronts on a compute unit nothing else covers a wavefront's LDS reads, so it reads the fragments of
  // the next pair of slices before it multiplies one (the down projection of one token: 35 us without, 26 with).
  constexpr bool AHEAD = RING_BYTES == DEEP_RING;
  // Pairs of slices in the ring (all but the one or two in registers are in flight), an even number: what fits its LDS, what the
  // counter of loads in flight can tell apart (below 64), and no more than 128 registers of A.
  constexpr int D_LDS = RING_BYTES / (NF * 2048), D_COUNT = 63 / LOADS + 1, D_REGS = 16 / M;
  constexpr int D = (D_LDS < D_COUNT ? (D_LDS < D_REGS ? D_LDS : D_REGS) : (D_COUNT < D_REGS ? D_COUNT : D_REGS)) & ~1;
  static_assert(D >= (AHEAD ? 4 : 2), "the ring holds the pairs being read and multiplied and at least one in flight");
  const int lane = threadIdx.x & 63;
  const int lrow = lane & 15, kg = lane >> 4;
  // Weight fragments.  Row f of fragment b of a group of 32 columns is column 8 (f >> 2) + 4 b + (f & 3), so that a lane
  // of the (transposed) result tiles holds 8 consecutive columns; the blocked layout stores the rows in that order.
  const char* wp[NF];
  if (PACKED) {
    const int tile = EPI == EPI_SWIGLU ? n0 >> 7 : n0 >> 8;
    const int r0 = EPI == EPI_SWIGLU ? n0 & 127 : n0 & 255;
    const char* base = p.W0 + (int64_t)expert * p.w_expert_bytes + (int64_t)tile * p.nsl * SLICE;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      wp[f] = base + (r0 + (f & 1) * 16 + (EPI == EPI_SWIGLU && f >= 2 ? 128 : 0)) * 64 + lane * 16;
    }
  } else {
    // Loads bring whole 128-byte lines (a pair of slices) of 8 rows each: lane l the chunk (l % 8) ^ (l / 8) of fragment row
    // l / 8 (and, 16 columns further, of row 8 + l / 8).  In LDS a fragment row is 128 bytes, chunk c at position c ^ (row % 8).
    const int c = n0 + 8 * (lane >> 5) + ((lane >> 3) & 3);
#pragma unroll
    for (int f = 0; f < NF; ++f)
      wp[f] = (EPI == EPI_SWIGLU && f >= 2 ? p.W1 : p.W0) + (int64_t)expert * p.w_expert_bytes +
              (int64_t)(c + 4 * (f & 1)) * p.nsl * 64 + (((lane & 7) ^ (lane >> 3)) << 4);
  }
  const char* xp[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int64_t r = row0 + m * 16 + lrow;
    if (r >= row_end) r = row_end - 1;
    r = p.row_of ? (int64_t)p.row_of[r] : r + (int64_t)expert * p.x_expert_rows;
    xp[m] = p.X + r * p.x_row_bytes + kg * 16;
  }
  f32x4 acc[NF][M];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[f][m][v] = 0.f;

  const int n = p.nsl >> 1;                          // pairs of slices (K is a multiple of 64)
  bf16x8 w[2][2][NF], xv[D][2][M];
  typedef __attribute__((address_space(3))) char lds_char;
  typedef const __attribute__((address_space(1))) void* gptr_t;
  lds_char* const ring3 = (lds_char*)ring;
  // (past its last pair a wavefront re-reads that one: in bounds, and the number of loads in flight is always the same)
  auto fetch = [&](int slot, int i) {
    const int s = 2 * (i < n ? i : n - 1);
    // 1 KB per load: packed, a fragment of slice s + j; row-major, both slices of 8 rows of a fragment
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        __builtin_amdgcn_global_load_lds(
            (gptr_t)(wp[f] + (PACKED ? (int64_t)(s + j) * SLICE : (int64_t)s * 64 + (int64_t)j * 16 * p.nsl * 64)),
            (__attribute__((address_space(3))) void*)(ring3 + slot * (NF * 2048) + f * 2048 + j * 1024), 16, 0, STREAM ? 2 : 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int m = 0; m < M; ++m) xv[slot][u][m] = *(const bf16x8*)(xp[m] + (int64_t)(s + u) * 64);
  };
  // where a lane's 16 bytes of slice u of a fragment lie in the ring
  const int frag_at[2] = {PACKED ? lrow * 64 + ((kg ^ ((lrow >> 2) & 3)) << 4) : lrow * 128 + ((kg ^ (lrow & 7)) << 4),
                          PACKED ? 1024 + lrow * 64 + ((kg ^ ((lrow >> 2) & 3)) << 4) : lrow * 128 + (((4 + kg) ^ (lrow & 7)) << 4)};
  auto read = [&](int slot, int set) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int f = 0; f < NF; ++f) w[set][u][f] = *(const bf16x8*)(ring + slot * (NF * 2048) + f * 2048 + frag_at[u]);
  };
  auto multiply = [&](int slot, int set) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < M; ++m)
          acc[f][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[set][u][f], xv[slot][u][m], acc[f][m], 0, 0, 0);
  };
#pragma unroll
  for (int d = 0; d < D - 1; ++d) fetch(d, d);
  if (AHEAD) {
    wait_until_flying<(D - 2) * LOADS>();
    read(0, 0);
  }
  int i0 = 0;
  for (; i0 + D <= n; i0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      __builtin_amdgcn_sched_barrier(0);   // (the slot's last fragments have been read)
      fetch((d + D - 1) % D, i0 + d + D - 1);
      wait_until_flying<(AHEAD ? D - 2 : D - 1) * LOADS>();
      read((d + AHEAD) % D, (d + AHEAD) & 1);
      multiply(d, d & 1);
    }
  }
  // the last n % D pairs, all of them in flight
  const int rest = n - i0;
  auto last = [&](auto self, auto at) {
    constexpr int d = decltype(at)::value;
    if constexpr (d < D - 1) {
      if (d < rest) {
        if constexpr (!AHEAD || d < D - 2) {
          wait_until_flying<(AHEAD ? D - 3 - d : D - 2 - d) * LOADS>();
          read(d + AHEAD, (d + AHEAD) & 1);
        }
        multiply(d, d & 1);
        self(self, std::integral_constant<int, d + 1>{});
      }
    }
  };
  last(last, std::integral_constant<int, 0>{});
  __builtin_amdgcn_s_waitcnt(0x0070);    // the re-reads still in flight target this workgroup's LDS
  // Register v of lane l of tile (f, m): column n0 + 8 (l / 16) + 4 (f & 1) + v, row 16 m + l % 16.
  const int col = n0 + 8 * kg;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int64_t r = row0 + m * 16 + lrow;
    if (r >= row_end) continue;
    const int64_t cr = r + (int64_t)expert * p.c_expert_rows;
    bf16x2 o[4];
    if (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        f32x2 h;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const int b = c >> 1, v = 2 * (c & 1) + d;
          const float g = acc[b][m][v], u = acc[(NF >> 1) + b][m][v];
          h[d] = g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
        }
        o[c] = __builtin_convertvector(h, bf16x2);
      }
      *(u32x4*)((uint16_t*)p.C + cr * p.ldc + col) = __builtin_bit_cast(u32x4, o);
    } else {
      int64_t dest = -1;
      if (EPI == EPI_ROWSCALE_F32 && p.row_dest) dest = p.row_dest[r];
      if (EPI == EPI_STORE || dest >= 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const f32x2 h = {acc[c >> 1][m][2 * (c & 1)], acc[c >> 1][m][2 * (c & 1) + 1]};
          o[c] = __builtin_convertvector(h, bf16x2);
        }
        uint16_t* const row = EPI == EPI_STORE ? (uint16_t*)p.C + cr * p.ldc : p.direct_out + dest * p.ldc;
        *(u32x4*)(row + col) = __builtin_bit_cast(u32x4, o);
      } else {
        const float sc = p.row_scale[r];
        float* dst = (float*)p.C + cr * p.ldc + col;
        *(f32x4*)dst = sc * acc[0][m];
        *(f32x4*)(dst + 4) = sc * acc[1][m];
      }
    }
  }
}

// MMAX: groups of 16 rows that any tile of the launch can hold; a tile takes the smallest body that fits it.
template <int EPI, bool PACKED, int MMAX, int RING_BYTES>
__global__ __launch_bounds__(64 * waves_of(RING_BYTES)) void gemm_few_kernel(FewArgs p) {
  constexpr int WAVES = waves_of(RING_BYTES);
  __shared__ __attribute__((aligned(16))) char rings[WAVES][RING_BYTES];
  const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int n0 = ((int)blockIdx.x * WAVES + wave) * 32;
  if (n0 >= p.N) return;              // (wavefronts share nothing: no barrier follows)
  char* const ring = rings[wave];
  const int t = blockIdx.y;
  int expert;
  int64_t row0, row_end;
  bool stream = p.stream;
  if (p.tile_expert) {
    if (t >= *p.tiles_in_use) return;
    expert = p.tile_expert[t];
    row0 = p.tile_row0[t];
    row_end = p.seg_end[expert];
    // Weights that another tile of the expert reads too are left to the caches (160 tokens on two experts: 509 -> 440 us).
    if ((t > 0 && p.tile_expert[t - 1] == expert) || row_end > row0 + FEW_ROWS) stream = false;
  } else {
    expert = t / p.row_tiles;
    row0 = (int64_t)(t - expert * p.row_tiles) * FEW_ROWS;
    row_end = p.rows;
  }
  if (row_end > row0 + FEW_ROWS) row_end = row0 + FEW_ROWS;
  const int rows = (int)(row_end - row0);
#define MOEP_FEW_TILE(M)                                                                     \
  do {                                                                                       \
    if (stream) few_tile<EPI, PACKED, M, true, RING_BYTES>(p, n0, expert, row0, row_end, ring);  \
    else few_tile<EPI, PACKED, M, false, RING_BYTES>(p, n0, expert, row0, row_end, ring);          \
  } while (0)
  if (MMAX == 1 || rows <= 16) MOEP_FEW_TILE(1);
  else if (MMAX == 2 || rows <= 32) MOEP_FEW_TILE(MMAX < 2 ? 1 : 2);
  else MOEP_FEW_TILE(MMAX < 4 ? 1 : 4);
#undef MOEP_FEW_TILE
}

template <int EPI, bool PACKED, int RING_BYTES>
void launch_ring(const FewArgs& a, int mmax, dim3 grid, hipStream_t s) {
  const dim3 threads(64 * waves_of(RING_BYTES));
  if (mmax == 1) hipLaunchKernelGGL((gemm_few_kernel<EPI, PACKED, 1, RING_BYTES>), grid, threads, 0, s, a);
  else if (mmax == 2) hipLaunchKernelGGL((gemm_few_kernel<EPI, PACKED, 2, RING_BYTES>), grid, threads, 0, s, a);
  else hipLaunchKernelGGL((gemm_few_kernel<EPI, PACKED, 4, RING_BYTES>), grid, threads, 0, s, a);
}

template <int EPI, bool PACKED>
int launch(const FewArgs& a, int mmax, bool deep, dim3 grid, hipStream_t s) {
  if (deep) launch_ring<EPI, PACKED, DEEP_RING>(a, mmax, grid, s);
  else launch_ring<EPI, PACKED, RING>(a, mmax, grid, s);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace

int launch_gemm_few(const FewGemmArgs& g, hipStream_t s, const char* name) {
  if (g.K <= 0 || g.K % 64 || g.N <= 0 || g.N % 32) return fail(MOEP_EUNSUPPORTED, "%s: K=%d, N=%d must be multiples of 64 and 32", name, g.K, g.N);
  if (((uintptr_t)g.X | (uintptr_t)g.W0 | (uintptr_t)g.W1 | (uintptr_t)g.C | (uintptr_t)g.direct_out) & 15)
    return fail(MOEP_EUNSUPPORTED, "%s: operands must be 16-byte aligned", name);
  if (g.ldx % 8 || g.ldc % 8 || g.ldc < g.N) return fail(MOEP_EINVAL, "%s: bad leading dimension", name);
  const bool grouped = g.tile_expert != nullptr;
  if (grouped && (!g.tile_row0 || !g.seg_end || !g.tiles_in_use)) return fail(MOEP_EINVAL, "%s: incomplete tile map", name);
  if (g.epilogue == EPI_ROWSCALE_F32 && !g.row_scale) return fail(MOEP_EINVAL, "%s: row_scale is NULL", name);
  if (g.max_rows <= 0) return MOEP_OK;
  int cus = 0;
  if (int st = gemm_device_ready(&cus)) return st;
  FewArgs a = {};
  a.W0 = (const char*)g.W0; a.W1 = (const char*)g.W1;
  a.w_expert_bytes = g.packed ? (int64_t)packed_b_bytes(g.N, g.K, g.epilogue == EPI_SWIGLU) : (int64_t)g.N * g.K * 2;
  a.X = (const char*)g.X; a.x_row_bytes = g.ldx * 2; a.row_of = g.row_of; a.x_expert_rows = g.x_expert_rows;
  a.C = g.C; a.ldc = g.ldc; a.c_expert_rows = g.c_expert_rows;
  a.N = g.N; a.nsl = g.K / 32;
  a.tile_expert = g.tile_expert; a.tile_row0 = g.tile_row0; a.seg_end = g.seg_end; a.tiles_in_use = g.tiles_in_use;
  a.row_tiles = (int)ceil_div(g.max_rows, FEW_ROWS); a.rows = g.max_rows;
  a.row_scale = g.row_scale; a.row_dest = g.row_dest; a.direct_out = (uint16_t*)g.direct_out;
  const int64_t tiles = grouped ? g.max_tiles : (int64_t)a.row_tiles * g.experts;
  if (tiles > 65535) return fail(MOEP_EUNSUPPORTED, "%s: too many tiles", name);
  const int units = g.N / 32;
  const int rows = (int)(g.max_rows < FEW_ROWS ? g.max_rows : FEW_ROWS);
  const int mmax = rows <= 16 ? 1 : rows <= 32 ? 2 : 4;
  // Few wavefronts (the expected tiles, a wavefront per 32 columns): the deep ring.
  const bool deep = (int64_t)units * (grouped ? g.busy_tiles : tiles) <= (int64_t)DEEP_WAVES * cus;
  // Weights far beyond the caches are read with the non-temporal hint, a layer that may still be cached is not.
  // Non-temporal against plain, forward: Mixtral shape, 16 tokens, packed 440 / 489 us, row-major 526 / 573; E 8, H 1024,
  // F 3584 (176 MB in all), 16 tokens, called again and again: 52 / 49.
  a.stream = (double)g.N * g.K * 2.0 * (g.epilogue == EPI_SWIGLU ? 2.0 : 1.0) * (grouped ? (double)g.busy_tiles : (double)g.experts) > STREAM_BYTES;
  const dim3 grid((unsigned)ceil_div(units, waves_of(deep ? DEEP_RING : RING)), (unsigned)tiles);
  Timed t(name, s);
  if (g.packed) {
    switch (g.epilogue) {
      case EPI_STORE: return launch<EPI_STORE, true>(a, mmax, deep, grid, s);
      case EPI_SWIGLU: return launch<EPI_SWIGLU, true>(a, mmax, deep, grid, s);
      default: return launch<EPI_ROWSCALE_F32, true>(a, mmax, deep, grid, s);
    }
  }
  switch (g.epilogue) {
    case EPI_STORE: return launch<EPI_STORE, false>(a, mmax, deep, grid, s);
    case EPI_SWIGLU: return launch<EPI_SWIGLU, false>(a, mmax, deep, grid, s);
    default: return launch<EPI_ROWSCALE_F32, false>(a, mmax, deep, grid, s);
  }
}

}  // namespace moep
