// Internal declarations shared by the host API and the kernel launchers of libmoeprune.
// Nothing here is part of the C ABI (that is include/moeprune.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "enum_plan.h"
#include "moeprune.h"
#include "skip_plan.h"
#include "tile_plan.h"

namespace moep {

// ---- errors -----------------------------------------------------------------
int fail(int status, const char* fmt, ...);   // records the thread's message, returns status

#define MOEP_HIP(expr)                                                                  \
  do {                                                                                  \
    hipError_t _e = (expr);                                                             \
    if (_e != hipSuccess)                                                               \
      return ::moep::fail(MOEP_EHIP, "%s failed: %s", #expr, hipGetErrorString(_e));    \
  } while (0)

// ---- per-kernel timing ------------------------------------------------------
// A Timed object brackets the launches made during its lifetime with a pair of
// HIP events on `stream` when timing is enabled; otherwise it does nothing.
struct Timed {
  Timed(const char* kernel_name, hipStream_t stream);
  ~Timed();
  int slot;
  hipStream_t stream;
};

static inline size_t align256(size_t n) { return (n + 255) & ~size_t(255); }
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t dtype_size(moep_dtype dt) { return dt == MOEP_BF16 ? 2 : 4; }

// ---- one token's logits -------------------------------------------------------
// Row t of logits [T,E] in registers, EMAX >= E (entries beyond E are 0), all loads in flight together; 16 bytes each when
// `vec` says that every row is 16-byte aligned.  A loop that loads and compares expert by expert waits for each load.
template <int EMAX>
__device__ __forceinline__ void load_logits(const float* __restrict__ logits, int64_t t, int E, bool vec, float (&v)[EMAX]) {
  const float* l = logits + t * E;
  if (vec) {
#pragma unroll
    for (int q = 0; q < EMAX / 4; ++q) {
      float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
      if (4 * q < E) f = *(const float4*)(l + 4 * q);
      v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < EMAX; ++e) v[e] = e < E ? l[e] : 0.f;
  }
}
static inline bool logits_vec(const float* logits, int E) { return E % 4 == 0 && ((uintptr_t)logits & 15) == 0; }

// The two largest logits among the kept experts (at least two); strict comparisons: the lower index wins a tie.
struct TopTwo { int e0, e1; float l0, l1; };
template <int EMAX>
__device__ __forceinline__ TopTwo top_two(const float (&v)[EMAX], int E, uint32_t kept) {
  int e0 = -1, e1 = -1;
  float l0 = 0.f, l1 = 0.f;
#pragma unroll
  for (int e = 0; e < EMAX; ++e) {
    const bool there = e < E && ((kept >> e) & 1u);   // a removed expert and its routing weight are gone
    const bool first = there && (e0 < 0 || v[e] > l0);
    const bool second = there && !first && (e1 < 0 || v[e] > l1);
    l1 = first ? l0 : second ? v[e] : l1;
    e1 = first ? e0 : second ? e : e1;
    l0 = first ? v[e] : l0;
    e0 = first ? e : e0;
  }
  return {e0, e1, l0, l1};
}

// ---- fp32 GEMM: C = epilogue(A B^T), A [M,K] and B [N,K] both K-contiguous, row-major operands -----
enum GemmEpilogue {
  EPI_STORE = 0,      // C[m,n] = acc                       (C in dt, N columns)
  EPI_SWIGLU = 1,     // C[m,n] = silu(A B0^T) * (A B1^T)    (C in dt, N columns)
  EPI_ROWSCALE_F32 = 2  // C[m,n] = row_scale[m] * acc        (C in fp32)
};

struct GemmArgs {
  const void* A = nullptr;       // [rows, K], leading dimension lda (elements)
  int64_t lda = 0;
  const int32_t* a_rows = nullptr;  // optional: logical row m reads A row a_rows[m]
  const void* B0 = nullptr;      // [N, K] (per expert), leading dimension K
  const void* B1 = nullptr;      // second weight for EPI_SWIGLU
  void* C = nullptr;             // [rows, N], leading dimension ldc (elements); 4-byte alignment suffices here and for C_rest
  int64_t ldc = 0;
  int64_t M = 0;                 // logical rows (dense mode) or upper bound on rows (grouped)
  int N = 0, K = 0;
  int epilogue = EPI_STORE;
  const float* row_scale = nullptr;
  // Grouped mode: rows seg_end[e - 1] (0) .. seg_end[e] - 1 are multiplied with expert e's weights, e < segments (0: dense).
  const int32_t* seg_end = nullptr;
  int segments = 0;
  int64_t b_expert_stride = 0;          // elements between consecutive experts' weights
  // Dense batched mode: `experts` GEMMs of the same shape in one launch.  Expert 0 reads A and writes C; expert e > 0
  // reads A_rest + (e - 1) a_expert_stride (A_rest NULL: A as well) and writes C_rest + (e - 1) c_expert_stride (elements).
  int experts = 1;
  const void* A_rest = nullptr;
  void* C_rest = nullptr;
  int64_t a_expert_stride = 0, c_expert_stride = 0;
  int busy_experts = 1;                 // grouped: experts that can have rows,
  bool rows_unknown = false;            //   and whether a threshold can leave them much fewer than M
};

constexpr int GEMM_BM = 256;   // rows per tile of the grouped map
// bf16 packed GEMM: M tiles per group of tiles that an XCD works through together, and output columns per tile,
// for the gate/up (SwiGLU) and the down projection (measured: the long-K down projection prefers 4 x 8 tiles per XCD)
constexpr int GEMM_GROUP_M_SWIGLU = 8, GEMM_GROUP_M_STORE = 4;
// output columns per tile; half-width tiles for launches that would leave compute units without a tile
constexpr int GEMM_BN_SWIGLU = 128, GEMM_BN_STORE = 256;
static inline int gemm_tile_columns(bool gate_up, bool half) { return (gate_up ? GEMM_BN_SWIGLU : GEMM_BN_STORE) >> (half ? 1 : 0); }
// 16-row groups that a wavefront multiplies in a launch whose tallest tile has `rows` rows: 8 (256 rows), 6 or 4
__host__ __device__ static inline int gemm_row_groups(int64_t rows) { return rows <= 128 ? 4 : rows <= 192 ? 6 : 8; }
// A tile order starts with a header: how many of its entries are full-width tiles, how many half-width ones (these come after
// the others), and the launch's row groups.
constexpr int TILE_ORDER_HEADER = 4, TILE_ORDER_HALF = 0, TILE_ORDER_ROW_GROUPS = 1, TILE_ORDER_FULL = 2;

int launch_gemm_f32(const GemmArgs& g, hipStream_t s, const char* name);

// ---- bf16 GEMM on packed operands (dense expert pass) ---------------------------------
// Operands are re-laid out once into 16 KB blocks of 256 rows x 32 k-values (the layout is described in
// gemm_bf16_packed.hip); EPI_SWIGLU writes its result as a packed A operand with K = N.
struct PackedGemmArgs {
  const void* A = nullptr;       // packed A operand, indexed by M tile
  const void* B = nullptr;       // packed_b_bytes(N, K, epilogue == EPI_SWIGLU) per expert
  bool b_row_major = false;      // B (and B1, the linear branch of EPI_SWIGLU) as the caller stores them: [N, K] per expert
  const void* B1 = nullptr;
  void* C = nullptr;             // EPI_STORE / EPI_ROWSCALE_F32: row-major [rows, ldc]; EPI_SWIGLU: packed A operand, K = N
  int64_t ldc = 0;
  int64_t M = 0;                 // rows (dense mode)
  int N = 0, K = 0;
  int epilogue = EPI_STORE;
  const float* row_scale = nullptr;
  // Grouped mode: M tile t covers rows tile_row0[t] .. of expert tile_expert[t] (< 0: no work), up to its segment's end; A (and a
  // packed C) hold one 256-row block per TILE.
  const int32_t* tile_expert = nullptr;
  const int32_t* tile_row0 = nullptr;
  const int32_t* seg_end = nullptr;
  int64_t max_m_tiles = 0;
  // Grouped mode: the order in which the launch walks its tiles: TILE_ORDER_HEADER words, then entry i = (M tile << 12) |
  // N tile (see write_order in skip.hip).
  const uint32_t* tile_order = nullptr;
  // Dense batched mode: `experts` GEMMs of the same shape in one launch; expert e reads A + e a_expert_bytes
  // (0: every expert reads the same A), B + e packed_b_bytes(..), and writes C + e c_expert_bytes.
  int experts = 1;
  bool stream = false;           // grouped: the weights that can be read are far more than the caches hold (routed_weights_stream)
  int64_t a_expert_bytes = 0, c_expert_bytes = 0;
  // EPI_ROWSCALE_F32, optional: rows r with row_dest[r] >= 0 are not written to C but, rounded to bf16 and
  // unscaled (their scale is 1), to row row_dest[r] of `direct_out` (leading dimension ldc): the slots of
  // tokens that were routed to a single expert go straight to the layer output.
  const int32_t* row_dest = nullptr;
  void* direct_out = nullptr;
};
size_t packed_a_bytes(int64_t rows, int K);
size_t packed_b_bytes(int N, int K, bool gate_up_pair);
int launch_pack_a_bf16(const void* X, int64_t ld, int64_t rows, int K, void* dst, hipStream_t s, const char* name);
// grouped: block row p of tile t = row rows_of[tile_row0[t] + p] of X
int launch_pack_a_gathered_bf16(const void* X, int64_t ld, const int32_t* rows_of, const int32_t* tile_expert,
                                const int32_t* tile_row0, const int32_t* seg_end, const int32_t* tiles_in_use,
                                const uint32_t* tile_order, int64_t max_tiles, int K, void* dst, hipStream_t s, const char* name);
// W1 != nullptr: gate/up pair (blocks of 128 rows of W0 followed by the same 128 rows of W1); `experts`
// consecutive [N, K] matrices are packed into consecutive packed_b_bytes blocks
int launch_pack_b_bf16(const void* W0, const void* W1, int N, int K, int experts, void* dst, hipStream_t s,
                       const char* name);
int launch_gemm_bf16_packed(const PackedGemmArgs& g, hipStream_t s, const char* name);

// ---- bf16 GEMM for few rows per expert (gemm_few.hip) -----------------------------------
constexpr int FEW_ROWS = 64;     // rows per tile of its grouped map
// Up to this many rows per expert the read of the weights bounds the layer and gemm_few.hip is the faster path; beyond
// it its 64-row tiles read A and the weights from the caches too often.  Dense calls: exactly; routed calls: on average, a
// token's k slots spread over the kept experts and none skipped.  Few-rows path against 256-row tiles, us per call:
// Mixtral shape (E 8, H 4096, F 14336), top-2, packed, T = 200 / 256 (50 / 64 rows): 639 / 691 against 679 / 676, row-major
// 710 / 762 against 817 / 816; dense, row-major, 48 rows 764 against 904, packed, 64 rows 782 against 695;
// layer of E 16, H 2048, F 5632, dense, packed, 32 / 64 rows: 309 / 414 against 376 / 381.
constexpr int64_t FEW_MAX_AVERAGE = 48;
// Routing need not be even: at worst all T tokens are on the same k experts, and each of those walks its weights once per
// 64 of them.  Beyond two such tiles the path is therefore kept to a lower average, unless the weights of k experts stay in
// the caches between the tiles (and T within eight of them).  All tokens on two experts, packed, us, few-rows path against
// 256-row tiles after packing or gathering x, evenly routed in brackets: Mixtral shape (705 MB for two experts) T = 128: 342
// against 415 (537 against 738), T = 160: 440 against 420 (608 against 742), T = 192: 533 against 424; E 8, H 1024, F 3584
// (44 MB) T = 160: 52 against 122 (56 against 117); E 32, H 2048, F 2048 (50 MB) T = 512: 112 against 149 (200 against 273),
// T = 640: 187 against 151 (221 against 270).
constexpr int64_t FEW_MAX_AVERAGE_MANY = 32;
constexpr double FEW_CACHED_BYTES = 128e6;   // (half of the last-level cache)
// k slots for each of T tokens, expert_bytes of weights per expert
inline bool few_rows(int64_t T, int k, int kept_experts, double expert_bytes) {
  if (k * T > FEW_MAX_AVERAGE * kept_experts) return false;
  return T <= 2 * FEW_ROWS || k * T <= FEW_MAX_AVERAGE_MANY * kept_experts || (T <= 8 * FEW_ROWS && k * expert_bytes <= FEW_CACHED_BYTES);
}
struct FewGemmArgs {
  const void* X = nullptr;       // row-major rows of A, leading dimension ldx
  int64_t ldx = 0;
  const int32_t* row_of = nullptr;   // grouped, optional: row r of the launch is row row_of[r] of X
  int64_t x_expert_rows = 0;     // dense: rows between consecutive experts of X (0: every expert reads the same rows)
  const void* W0 = nullptr;      // packed: blocked copy of every expert's weights; else [experts, N, K] row-major
  const void* W1 = nullptr;      // row-major EPI_SWIGLU: the linear branch
  bool packed = false;
  void* C = nullptr;             // EPI_STORE, EPI_SWIGLU: bf16 rows; EPI_ROWSCALE_F32: fp32 rows; leading dimension ldc
  int64_t ldc = 0, c_expert_rows = 0;
  int N = 0, K = 0;
  int epilogue = EPI_STORE;
  int64_t max_rows = 0;          // dense: rows; grouped: most rows an expert can have
  int64_t busy_tiles = 1;        // tiles that are expected to hold rows (choose the load ring and the cache policy)
  int experts = 1;               // dense
  // grouped: the tile map of PackedGemmArgs with FEW_ROWS rows per tile
  const int32_t* tile_expert = nullptr;
  const int32_t* tile_row0 = nullptr;
  const int32_t* seg_end = nullptr;
  const int32_t* tiles_in_use = nullptr;
  int64_t max_tiles = 0;
  const float* row_scale = nullptr;
  const int32_t* row_dest = nullptr;   // as in PackedGemmArgs
  void* direct_out = nullptr;
};
int launch_gemm_few(const FewGemmArgs& g, hipStream_t s, const char* name);
// First use of a device by a bf16 expert GEMM: raises the dynamic LDS limits of all of them; its compute-unit count.
int gemm_device_ready(int* compute_units);

// ---- router -------------------------------------------------------------------
int launch_router(const void* x, const void* Wgate, int64_t T, int E, int H, moep_dtype dt,
                  float* logits, hipStream_t s);
// bf16: the same logits (bit for bit) and the packed A-operand copy of x in one pass; MOEP_EUNSUPPORTED, with nothing
// launched and no message, for shapes without a fused kernel
int launch_router_and_pack_x(const void* x, const void* Wgate, int64_t T, int E, int H, float* logits, void* xpacked,
                             hipStream_t s);

// ---- enumeration ----------------------------------------------------------------
// Expert outputs of the rank-limited pass: row slot_of[t, j] of Y is the output of expert
// experts[t, j], the token's j-th ranked expert, j < n_rank.
struct RankedSource {
  const int32_t* slot_of;
  const int32_t* experts;
  int n_rank;
};
// One r, and where its results go.
struct EnumJob {
  EnumPlan plan;
  float* loss; int32_t* argmin; uint32_t* argmin_mask; int64_t* unaffected;   // unaffected may be NULL
};
// Every job on the same logits and Y, up to RECORD_SETS of them; ws_bytes: the largest of their plans' totals.
int launch_enumerate(const EnumJob* jobs, int n, const float* logits, const void* Y, moep_dtype dt, char* ws, size_t ws_bytes,
                     hipStream_t s, const RankedSource* ranked = nullptr);
// One job through Gram matrices at the start of the workspace (reuse_gram: they are there already, from another r).
int launch_enumerate_from_gram(const EnumJob& job, const float* logits, const void* Y, moep_dtype dt, char* ws, hipStream_t s,
                               const RankedSource* ranked, bool reuse_gram);

// fp64 sum of n_tiles partial sums per subset (partial[tile * n_sub + subset]) in a fixed order -> loss; sum of the
// partial counts (NULL: *unaffected holds it already) -> *unaffected (may be NULL; `cleared`: already 0); lowest-index argmin and its kept mask
int launch_reduce_argmin(const float* partial, const uint32_t* partial_cnt, int64_t n_tiles, int64_t n_sub, int E,
                         int r, float* loss, int32_t* argmin, uint32_t* argmin_mask, int64_t* unaffected, bool cleared,
                         hipStream_t s);
// masks[i] = kept mask of subset i
int launch_subset_masks(int E, int r, int64_t n_sub, uint32_t* masks, hipStream_t s);

// The same losses straight from the definition, without Gram matrices (enumerate_direct.hip).
struct DirectPlan {
  int64_t T; int E, H, k, r;
  int64_t n_sub;
  int blocks;        // workgroups, each walking tokens b, b + blocks, ...
  size_t lds_bytes;  // dynamic LDS per workgroup
  size_t off_masks, off_partial, off_partial_cnt, total;
};
int plan_enumerate_direct(int64_t T, int E, int H, int k, int r, moep_dtype dt, DirectPlan* p);
int launch_enumerate_direct(const DirectPlan& p, const float* logits, const void* Y, moep_dtype dt, float* loss,
                            int32_t* argmin, uint32_t* argmin_mask, int64_t* unaffected, char* ws, hipStream_t s);

// ---- skipping ---------------------------------------------------------------------
// Whether the routing of a handful of tokens computes their logits as well, in the same launch: it is then given x and Wgate
// (both NULL otherwise) and writes `logits`.
bool routing_computes_logits(const SkipPlan& p, const void* x, const void* Wgate);
int launch_skip_routing(const SkipPlan& p, const float* logits, uint32_t kept_mask, float beta, uint8_t* skip_mask,
                        int32_t* top2_out, char* ws, hipStream_t s, const void* x = nullptr, const void* Wgate = nullptr);
// `singles_done`: tokens routed to a single expert already have their output (written by the down projection)
int launch_skip_combine(const SkipPlan& p, moep_dtype dt, const uint8_t* skip_mask, void* out,
                        char* ws, hipStream_t s, bool singles_done);
int launch_skip_topk_routing(const SkipPlan& p, const float* logits, uint32_t kept_mask, float beta,
                             int32_t* n_used, int32_t* topk_out, char* ws, hipStream_t s,
                             int32_t* pos_out = nullptr, const void* x = nullptr, const void* Wgate = nullptr);
int launch_skip_topk_combine(const SkipPlan& p, moep_dtype dt, void* out, char* ws, hipStream_t s, bool singles_done);

// ---- beta calibration -----------------------------------------------------------------
size_t calibrate_workspace_bytes(int64_t T);
int launch_calibrate_beta(const float* logits, int64_t T, int E, uint32_t kept_mask, float* beta_out,
                          char* ws, hipStream_t s);

// ---- selection statistics ---------------------------------------------------------------
int launch_selection_stats(const float* logits, int64_t T, int E, int k, int r, int64_t* count, int64_t* co,
                           uint32_t* freq_mask, hipStream_t s);

// Host-side subset helpers (also used to fill the device mask table).
int64_t binomial(int n, int r);
uint32_t unrank_mask(int E, int r, int64_t idx);

}  // namespace moep
