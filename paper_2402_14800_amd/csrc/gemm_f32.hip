// fp32 GEMM (storage type MOEP_F32): C = epilogue(A B^T) on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 accumulate).  Serves layers kept in fp32; the layout of arguments and the epilogues are those of the
// bf16 kernel.
//
// Bound by the fp32 matrix rate (157 TFLOP/s nominal; 109 reached at 6000 tokens) where there are tiles for the chip, by the
// serial walk over K where there are not.  A workgroup of 256 threads owns 64 rows x 128 accumulator columns (gate/up: 64
// columns of either branch; few tiles: 32 x 128, then 32 x 64) and walks K in slabs of 32 through a ring of LDS stages that
// direct loads fill one or two slabs ahead, one barrier per slab (how many: f32_slabs_ahead in tile_plan.h).  Against a slab in
// registers and two buffers, all experts, E 8, H 512, F 1024: T = 64 164 -> 145 us, 400 226 -> 208, 1501 453 -> 434, 4000 973 ->
// 936, 6000 1379 -> 1369; E 4, H 1024, F 3584, T = 400 514 -> 466.  The tiles are small because the layers are: a dense pass takes as
// many experts per launch as its scratch room allows for the same reason.
// A row of a slab is 128 bytes in LDS, its 16-byte chunk c at position c ^ (row & 7), so that the fragment reads (16 rows
// apart 128 bytes) are free of bank conflicts.  A lane reads 4 consecutive k as one 16-byte word; element j of it feeds
// MFMA j, for both operands alike, so the four MFMAs of 16 k-values sum k = j, 4 + j, 8 + j, 12 + j.
// Measured, all experts, E 8, H 512, F 1024, against the plain-FMA kernel with 64 x 64 tiles that this replaces: T = 64
// 1356 -> 145 us, 1501 1369 -> 434, 6000 2284 -> 1369; E 4, H 64, F 128, T = 512: 109 -> 36 us.
// A row's sum depends on K only, so a token's outputs do not depend on the batch or on the tile.
#include "common.h"

namespace moep {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int TK = 32, THREADS = 256;                      // k per slab

struct FArgs {
  const float* A; const float* B0; const float* B1;
  const int32_t* a_rows;
  float* C;
  const float* row_scale;
  const int32_t* seg_end; int segments;                    // routed: the experts' segment ends; segments 0: dense
  int64_t M, lda, ldc, b_expert_stride;
  const float* A_rest; float* C_rest;                      // dense, blockIdx.z = expert: experts 1, 2, ...
  int64_t a_expert_stride, c_expert_stride;
  int N, K;
  bool c_by_word;                                          // C or C_rest is not 16-byte aligned: stored float by float
  bool by_register;                                        // the weights are not 16-byte aligned
  bool columns_first;                                      // blockIdx.x walks the column tiles, y the row tiles
};

template <int EPI, int TM, int TB, int AHEAD>    // TM = rows, TB = accumulator columns per tile; AHEAD = slabs in flight
__global__ __launch_bounds__(THREADS) void gemm_f32_kernel(FArgs p) {
  constexpr int RT = TM / 32, CT = TB / 32;                // 16-row and 16-column tiles of a wavefront = rows staged per thread
  constexpr int SLAB = (TM + TB) * TK;                     // floats of one LDS stage
  constexpr int LOADS = (TM + TB) / 32;                    // 1 KB loads of a wavefront per slab
  constexpr int TN = EPI == EPI_SWIGLU ? TB / 2 : TB;      // output columns
  __shared__ __attribute__((aligned(16))) float lds[AHEAD + 1][SLAB];

  const unsigned row_tile = p.columns_first ? blockIdx.y : blockIdx.x, column_tile = p.columns_first ? blockIdx.x : blockIdx.y;
  int64_t row0, row_end;
  int64_t expert = blockIdx.z;
  if (p.segments) {
    // The experts' tiles of TM rows one after the other, lane e holding expert e's, so that the row tiles without rows are the last ones
    // of the grid.  Workgroups are dealt to the compute units in turn, whichever of them return at once: from a map of 256-row tiles,
    // whose first TM-row part always has rows and whose last often has none, the first parts met on the same compute units and some of
    // these had a round more.  us per call, nothing skipped, from the map / so: E 16, H 1024, F 512, T = 2000 215 / 213, 2500 288 / 217,
    // 2750 337 / 218; E 4, H 1472, F 1908, T = 244 201 / 128; launches of 10 us are up to 0.5 us longer (E 8, H 156, F 96, top-3,
    // T = 2594 42.1 / 43.4).
    const int l = threadIdx.x & 63;
    const int end = l < p.segments ? p.seg_end[l] : 0;
    const int begin = __builtin_amdgcn_update_dpp(0, end, 0x138, 0xf, 0xf, true);            // the lane before (lane 0: 0)
    const int tiles = l < p.segments ? (int)(((unsigned)(end - begin) + TM - 1) / TM) : 0;
    int through = tiles;                                   // tiles of the experts up to this lane's: sums over 16 lanes,
    through += __builtin_amdgcn_update_dpp(0, through, 0x111, 0xf, 0xf, true);
    through += __builtin_amdgcn_update_dpp(0, through, 0x112, 0xf, 0xf, true);
    through += __builtin_amdgcn_update_dpp(0, through, 0x114, 0xf, 0xf, true);
    through += __builtin_amdgcn_update_dpp(0, through, 0x118, 0xf, 0xf, true);
    through += __builtin_amdgcn_update_dpp(0, through, 0x142, 0x2, 0xf, false);              // and the first 16 to the second
    const int e = __popcll(__ballot(l < p.segments && through <= (int)row_tile));
    if (e >= p.segments) return;
    expert = e;
    row_end = __builtin_amdgcn_readlane(end, e);
    row0 = __builtin_amdgcn_readlane(begin, e) + (int64_t)((int)row_tile - __builtin_amdgcn_readlane(through - tiles, e)) * TM;
  } else {
    row0 = (int64_t)row_tile * TM;
    row_end = p.M;
  }
  const float* const A = blockIdx.z && p.A_rest ? p.A_rest + (blockIdx.z - 1) * p.a_expert_stride : p.A;
  float* const C = blockIdx.z ? p.C_rest + (blockIdx.z - 1) * p.c_expert_stride : p.C;
  const float* const B0 = p.B0 + expert * p.b_expert_stride;
  const float* const B1 = EPI == EPI_SWIGLU ? p.B1 + expert * p.b_expert_stride : nullptr;
  const int n0 = column_tile * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // staging: a load brings 8 rows, lane l the chunk that belongs at position l % 8 of row l / 8; wavefront w the rows 8 w .. + 7 of
  // every 32 of A, then of B.  Rows beyond the last one repeat it (their products are not stored).
  const int sr = tid >> 3, sc = (tid & 7) ^ (sr & 7);
  const float* src[LOADS];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    int64_t r = row0 + sr + 32 * i;
    if (r >= row_end) r = row_end - 1;
    src[i] = A + (p.a_rows ? (int64_t)p.a_rows[r] : r) * p.lda + sc * 4;
  }
#pragma unroll
  for (int i = 0; i < CT; ++i) {
    const int br = sr + 32 * i;
    const float* base = EPI == EPI_SWIGLU && br >= TN ? B1 : B0;
    int n = n0 + (EPI == EPI_SWIGLU ? br % TN : br);
    if (n >= p.N) n = p.N - 1;
    src[RT + i] = base + (int64_t)n * p.K + sc * 4;
  }
  typedef __attribute__((address_space(3))) char lds_char;
  lds_char* const lds3 = (lds_char*)&lds[0][0] + __builtin_amdgcn_readfirstlane(wave) * 1024;
  const int slabs = p.by_register ? 0 : p.K / TK;          // whole ones
  auto fetch = [&](int stage, int slab) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + slab * TK),
                                       (__attribute__((address_space(3))) void*)(lds3 + stage * (SLAB * 4) + i * 4096), 16, 0, 0);
  };

  const int frow = lane & 15, fg = lane >> 4;
  f32x4 acc[RT][CT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto multiply = [&](const float* buf) {
#pragma unroll
    for (int h = 0; h < TK / 16; ++h) {
      const int pos = ((4 * h + fg) ^ (frow & 7)) << 2;    // (fragment rows are 16 apart: the same position in all)
      f32x4 fa[RT], fb[CT];
#pragma unroll
      for (int i = 0; i < RT; ++i) fa[i] = *(const f32x4*)(buf + (wm * (TM / 2) + i * 16 + frow) * TK + pos);
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        const int r = EPI == EPI_SWIGLU ? (j / (CT / 2)) * TN + wn * (TN / 2) + (j % (CT / 2)) * 16 : wn * (TB / 2) + j * 16;
        fb[j] = *(const f32x4*)(buf + TM * TK + (r + frow) * TK + pos);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < CT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
    }
  };
  // Slab s + AHEAD goes into the stage of slab s - 1, which every wavefront has read when it meets the others in front of slab s.
  // Past the last whole slab a wavefront re-reads that one (in bounds, into a stage nobody reads again), so that the loads in
  // flight are the same in every step.
  if (slabs > 0) {
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) fetch(s, s < slabs ? s : slabs - 1);
    int stage = 0, next = AHEAD;
    for (int s = 0; s < slabs; ++s) {
      __builtin_amdgcn_sched_barrier(0);
      constexpr int FLYING = (AHEAD - 1) * LOADS;          // of the slabs after this one
      __builtin_amdgcn_s_waitcnt(0x0070 | (FLYING & 15) | ((FLYING >> 4) << 14));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      fetch(next, s + AHEAD < slabs ? s + AHEAD : slabs - 1);
      multiply(lds[stage]);
      stage = stage == AHEAD ? 0 : stage + 1;
      next = next == AHEAD ? 0 : next + 1;
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070);                    // the re-reads target this workgroup's LDS
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  // A last slab that is not whole (K is a multiple of 4: chunks beyond it are zero), and every slab of weights that are not
  // 16-byte aligned, goes through registers, into two of the stages in turn.
  f32x4 held[LOADS];
  auto hold = [&](int slab) {
    const bool in = slab * TK + sc * 4 < p.K;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) held[i] = in ? *(const f32x4*)(src[i] + slab * TK) : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  if (slabs * TK < p.K) hold(slabs);
  for (int s = slabs; s * TK < p.K; ++s) {
    float* const buf = lds[(s - slabs) & 1];               // (last read before the previous barrier)
#pragma unroll
    for (int i = 0; i < LOADS; ++i) *(f32x4*)(buf + tid * 4 + i * 1024) = held[i];
    __syncthreads();
    if ((s + 1) * TK < p.K) hold(s + 1);
    multiply(buf);
  }

  // Register v of lane l of tile (i, j): row 16 i + l % 16 of the wavefront's TM / 2, weight row 4 (l / 16) + v of tile j.
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int64_t r = row0 + wm * (TM / 2) + i * 16 + frow;
    if (r >= row_end) continue;
    const float scale = EPI == EPI_ROWSCALE_F32 ? p.row_scale[r] : 1.0f;
#pragma unroll
    for (int j = 0; j < (EPI == EPI_SWIGLU ? CT / 2 : CT); ++j) {
      const int n = n0 + wn * (TN / 2) + j * 16 + fg * 4;
      if (n >= p.N) continue;                              // N is a multiple of 4
      f32x4 o;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float x = acc[i][j][v];
        if (EPI == EPI_SWIGLU) x = x / (1.0f + expf(-x)) * acc[i][CT / 2 + j][v];
        if (EPI == EPI_ROWSCALE_F32) x *= scale;
        o[v] = x;
      }
      float* const dst = C + r * p.ldc + n;
      if (p.c_by_word) {
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[v] = o[v];
      } else {
        *(f32x4*)dst = o;
      }
    }
  }
}

// (two 64-row tiles per compute unit; T 1501 of the layer above: 470 us with the line at 512 tiles, 551 us without 32-row tiles)
constexpr int64_t SMALL_TILES_BELOW = 512;
// (the same line for half the width again: T 64 of that layer 241 -> 164 us, 400 270 -> 227, 1501 470 -> 454; at 256 tiles 464)
constexpr int64_t NARROW_TILES_BELOW = 512;

}  // namespace

int launch_gemm_f32(const GemmArgs& g, hipStream_t s, const char* name) {
  if (g.K % 4 || g.K <= 0 || g.lda % 4) return fail(MOEP_EUNSUPPORTED, "%s: K=%d and lda must be multiples of 4", name, g.K);
  if (g.N % 4 || g.ldc % 4) return fail(MOEP_EUNSUPPORTED, "%s: N=%d and ldc must be multiples of 4", name, g.N);
  if (g.M <= 0 || g.N <= 0) return MOEP_OK;
  FArgs f = {};
  f.A = (const float*)g.A; f.B0 = (const float*)g.B0; f.B1 = (const float*)g.B1;
  f.a_rows = g.a_rows; f.C = (float*)g.C; f.row_scale = g.row_scale;
  f.seg_end = g.seg_end; f.segments = g.segments;
  f.M = g.M; f.lda = g.lda; f.ldc = g.ldc; f.b_expert_stride = g.b_expert_stride;
  f.A_rest = (const float*)g.A_rest; f.C_rest = (float*)g.C_rest;
  f.a_expert_stride = g.a_expert_stride; f.c_expert_stride = g.c_expert_stride;
  f.N = g.N; f.K = g.K;
  const bool several = g.experts > 1;      // (the *_rest operands are of no use otherwise)
  if (((uintptr_t)g.A | (several ? (uintptr_t)g.A_rest : 0)) & 15) return fail(MOEP_EUNSUPPORTED, "%s: A must be 16-byte aligned", name);
  f.by_register = (((uintptr_t)g.B0 | (uintptr_t)g.B1) & 15) != 0;
  f.c_by_word = (((uintptr_t)g.C | (several ? (uintptr_t)g.C_rest : 0)) & 15) != 0;
  if (g.experts < 1 || g.experts > 65535 || (g.segments && g.experts != 1)) return fail(MOEP_EINVAL, "%s: bad batch count %d", name, g.experts);
  if (g.segments < 0 || g.segments > 32 || (g.segments && (!g.seg_end || g.M >= ((int64_t)1 << 31)))) return fail(MOEP_EINVAL, "%s: bad segments", name);
  // row tiles: for the choice between the forms, of a routed launch those of a map of 256-row tiles; and how many there can be
  auto m_tiles = [&](int tm) { return g.segments ? (ceil_div(g.M, GEMM_BM) + g.segments) * (GEMM_BM / tm) : ceil_div(g.M, tm); };
  auto n_tiles = [&](int tb) { return ceil_div(g.N, g.epilogue == EPI_SWIGLU ? tb / 2 : tb); };
  // 64 x 128 accumulators per tile, 32 x 128 where those are few, 32 x 64 where these are
  const int tm = m_tiles(64) * n_tiles(128) * g.experts < SMALL_TILES_BELOW ? 32 : 64;
  const int tb = tm == 32 && m_tiles(32) * n_tiles(128) * g.experts < NARROW_TILES_BELOW ? 64 : 128;
  // (weights that are not 16-byte aligned use two stages only: as many workgroups per compute unit as there can be; so it is with
  // rows that a threshold leaves, whose number is known on the device only: 70 routed layers of 200 to 8000 tokens with one, against
  // row tiles from the map, geometric mean and worst: one ahead 0.80, 1.01, two 0.80, 1.01, by the rule for all rows 0.80, 1.06)
  const int64_t tiles = (g.segments ? routed_row_tiles(g.M, g.busy_experts, tm) : ceil_div(g.M, tm)) * n_tiles(tb) * g.experts;
  const int ahead = (f.by_register && tiles > 512) || g.rows_unknown ? 1 : f32_slabs_ahead(tiles, 2, tm == 64 ? 3 : 4);
  const int64_t row_tiles = ceil_div(g.M, tm) + g.segments;
  if (row_tiles > 2147483647LL || n_tiles(tb) > GRID_Y_MAX) return fail(MOEP_EUNSUPPORTED, "%s: too many tiles", name);
  dim3 grid((unsigned)row_tiles, (unsigned)n_tiles(tb), (unsigned)g.experts);
  f.columns_first = f32_columns_first(g.segments > 0, row_tiles);
  if (f.columns_first) grid = dim3((unsigned)n_tiles(tb), (unsigned)row_tiles, 1);
  Timed t(name, s);
#define MOEP_F32_LAUNCH(EPI, TM, TB, AHEAD) hipLaunchKernelGGL((gemm_f32_kernel<EPI, TM, TB, AHEAD>), grid, dim3(THREADS), 0, s, f)
#define MOEP_F32_CASE(EPI)                                                                              \
  case EPI:                                                                                             \
    if (tb == 64) MOEP_F32_LAUNCH(EPI, 32, 64, 2);                                                      \
    else if (tm == 32 && ahead == 1) MOEP_F32_LAUNCH(EPI, 32, 128, 1);                                  \
    else if (tm == 32) MOEP_F32_LAUNCH(EPI, 32, 128, 2);                                                \
    else if (ahead == 1) MOEP_F32_LAUNCH(EPI, 64, 128, 1);                                              \
    else MOEP_F32_LAUNCH(EPI, 64, 128, 2);                                                              \
    break;
  switch (g.epilogue) {
    MOEP_F32_CASE(EPI_STORE) MOEP_F32_CASE(EPI_SWIGLU) MOEP_F32_CASE(EPI_ROWSCALE_F32)
    default: return fail(MOEP_EINVAL, "%s: unknown epilogue %d", name, g.epilogue);
  }
#undef MOEP_F32_CASE
#undef MOEP_F32_LAUNCH
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
