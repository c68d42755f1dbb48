// bf16 GEMM for gfx950 on PACKED operands: C = epilogue(A B^T), fp32 accumulate on the MFMA units
// (v_mfma_f32_16x16x32_bf16).  The bf16 expert GEMMs with more than a few dozen rows per expert
// (gemm_few.hip takes those with fewer): the dense pass (every expert on every
// token, Sec. 3.1 / Sec. 3.2) and, in grouped mode, the routed rows of the skipping forward (Sec. 3.3)
// and of the rank-limited pass.  The operands are re-read many times; re-laying them out once is
// almost free.
//
// Packed layout.  A matrix X [R, K] is cut into blocks of 256 rows x 32 k-values ("slices").  Block
// (row tile t, slice s) is 16 KB, stored contiguously at ((t * K/32) + s) * 16 KB; inside it row p
// takes 64 bytes and its four 16-byte chunks are permuted, chunk c at position c ^ ((p >> 2) & 3).
// That is exactly the image the kernel wants in LDS (fragment reads of 16 consecutive rows are then
// free of bank conflicts), so a wavefront's direct global->LDS load moves 1 KB of CONSECUTIVE bytes:
// eight full cache lines per instruction whatever K is, where the row-major layout offers 128-byte
// pieces one row pitch apart (or half lines, with 32-wide slices).
// Weight blocks carry two more permutations (see pack_kernel): the rows of every group of 32 are
// reordered so that the transposed accumulator tiles give each lane 8 consecutive output columns, and
// for the gate/up projection a block holds 128 rows of W1 followed by the same 128 rows of W3.
//
// BROW: the weight operand is read as the caller stores it, row-major, in whole 128-byte lines: a "unit" is half of the
// tile's weight rows (gate/up: the rows of one branch) over TWO slices, and a step loads one unit where it would load one
// slice of all rows; the row permutation is in the loads' lane addresses.  Half lines, one slice of all rows per step, had
// come at about 4 TB/s, fetched twice.  The same products in the same order, hence the same bits.  Skipping forward,
// Mixtral shape, T = 300 826 -> 697 us, 777 851 -> 712, 1500 1194 -> 1075, 6000 2886 -> 2710; 1 to 2 % slower than on
// packed weights where the matrix rate is the bound, without the packing pass.
//
// Kernel.  One workgroup of 256 threads (4 wavefronts, 2 along M x 2 along N, one per SIMD) owns a
// 256 x 256 tile of the accumulator (256 x 128 outputs in SwiGLU mode); a wavefront owns 128 x 128 =
// 8 x 8 MFMA tiles, whose 256 accumulator registers sit in the AGPR half of the wavefront's 512 registers.
// K is walked one slice (one MFMA depth) at a time through a ring of NS = 5 LDS stages of 32 KB.  In
// the step that multiplies slice g a wavefront also issues its 8 direct loads of slice g + NS - 1 (one
// per 6 MFMAs, into the stage whose fragments were read two steps ago) and reads the fragments of slice
// g + 1 into the other half of a double-buffered fragment register set: 64 MFMAs, 16 LDS reads and 8
// loads per step.  Loads are spread evenly over the step, never issued in bursts.  On blocked weights the
// wavefronts meet at a barrier every SECOND step only: before it each waits until all but the newest step's
// loads have landed, which covers the two slices read in the two steps that follow; the stage a step's loads
// overwrite was last read two steps earlier, i.e. before the previous barrier.  On row-major weights (BROW) there is a
// barrier after every step, since the second unit of a pair of slices is issued one step before it is read (wait counts
// at W_MAIN and W_ODD).  In a body of half width (NG = 4) or for short tiles (MG = 6 or 4) a wavefront's step has
// MG x NG MFMAs, MG + NG reads and (MG + NG) / 2 loads.
// Workgroups are persistent (one per compute unit) and the ring runs across tile boundaries: while the
// last slices of a tile are multiplied and its epilogue runs, the first slices of the workgroup's next
// tile are already being fetched.  The loader changes tile only BETWEEN runs of steps (a tile's steps
// are cut where the loader, NS - 1 slices ahead, reaches the end of its tile), so the hot loop is a
// single basic block of two steps with no tile bookkeeping in it; with a branch in the loop the
// register allocator moved accumulators between AGPRs and VGPRs on every step.
//
// The 32 workgroups of an XCD are kept in step, round of tiles by round of tiles, through a counter in
// device memory (bounded wait, see round_sync).
//
// Epilogues.  The MFMAs take the weight fragment as first operand, so an accumulator tile is the
// transpose of the output tile and (with the row permutation above) a lane holds 8 consecutive output
// columns of one row: one 16-byte store.  SwiGLU mode (Sec. 3.1) forms silu(gate) * up in registers,
// rounds once to bf16 and writes the result in the PACKED layout of an A operand with K = N, ready
// for the down projection: 16 rows x 64 bytes = 1 KB contiguous per wavefront store.
//
// Workgroup order: logical tile ids are dealt round-robin to the 8 XCDs (as the hardware deals
// workgroups) and remapped so that every XCD works on a contiguous run of tiles, GROUP_M M-tiles deep
// before moving along N, so that the 32 tiles in flight on one XCD share operand panels in its L2.
// Grouped launches read that order from a table the dispatch kernels lay out, with the groups of M tiles
// aligned to the experts' segments (a group that straddled two experts would share no weight panel).
#include <mutex>
#include <type_traits>

#include "common.h"

namespace moep {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;   // one 16-byte chunk

constexpr int THREADS = 256;
constexpr int SYNC_POLLS = 64;                // bound of a workgroup's wait for the others of its XCD
constexpr uint32_t SYNC_EVERY = 4;            // tiles between two line-ups (1: 0.9 % slower; the L2 hit rate is the same)
constexpr int NS = 5;                       // ring stages
constexpr int SLICE = 256 * 64;             // one operand block: 256 rows x 32 bf16
constexpr int RING = NS * SLICE;            // bytes of one operand's ring
constexpr int LDS_BYTES = 2 * RING;         // A's ring, then B's: 160 KB
static_assert(GEMM_BM == 256, "tiles are 256 rows");
static_assert((NS - 1) % 2 == 0, "the loader must be an even number of slices ahead (steps come in pairs)");

// LDS row p of a weight block holds weight row perm32(p) of the tile: inside every group of 32 rows,
// LDS row 16 b + f is weight row 8 (f >> 2) + 4 b + (f & 3).
__host__ __device__ constexpr int perm32(int p) {
  return (p & ~31) | ((p & 12) << 1) | ((p & 16) >> 2) | (p & 3);
}

// ---- packing ---------------------------------------------------------------------------------
// mode 0: A operand, block row p of tile t = source row 256 t + p.
// mode 1: weight, 256 output columns per tile: block row p = row 256 t + perm32(p) of W0.
// mode 2: gate/up weight pair, 128 output columns per tile: block row p < 128 = row 128 t + perm32(p) of
//         W0, block row p >= 128 = row 128 t + perm32(p - 128) of W1.
// mode 3: gathered A operand of a grouped GEMM: block row p of tile t = source row rows_of[tile_row0[t] + p]
//         (the rows routed to the tile's expert, Sec. 3.3); tiles beyond the number in use are left alone, and so are
//         the rows that the launch's bodies do not fetch (16 rows x 2 for each of tile_order's row groups).
// Rows beyond the last one re-read the last row (their products are never stored).
// One workgroup moves a pair of slices (64 k-values) of one tile, so that whole 128-byte lines are read;
// blockIdx.z selects the expert of a weight stack.
struct PackArgs {
  const u32x4* W0; const u32x4* W1;
  u32x4* dst;
  int64_t ld_chunks;      // source leading dimension in 16-byte chunks
  int64_t rows;           // valid source rows (modes 0..2)
  int64_t src_expert_chunks, dst_expert_chunks;   // per-expert strides (blockIdx.z)
  const int32_t* rows_of; const int32_t* tile_expert; const int32_t* tile_row0; const int32_t* seg_end;
  const int32_t* tiles_in_use; const uint32_t* tile_order;
  int nsl;                // K / 32
  int mode;
};

__global__ __launch_bounds__(256) void pack_kernel(PackArgs p) {
  const int t = blockIdx.x;
  const int sp = blockIdx.y;                 // slice pair
  const u32x4* W0 = p.W0 + (int64_t)blockIdx.z * p.src_expert_chunks;
  const u32x4* W1 = p.W1 + (int64_t)blockIdx.z * p.src_expert_chunks;
  u32x4* dst = p.dst + (int64_t)blockIdx.z * p.dst_expert_chunks;
  int64_t g_row0 = 0, g_end = 0;
  int groups = 8;
  if (p.mode == 3) {
    if (t >= *p.tiles_in_use) return;
    groups = (int)p.tile_order[TILE_ORDER_ROW_GROUPS];
    g_row0 = p.tile_row0[t];
    g_end = p.seg_end[p.tile_expert[t]];
  }
  auto move = [&](auto pieces) {             // of 32 rows; a loop of its own for each number, all its loads in flight together
#pragma unroll
    for (int it = 0; it < decltype(pieces)::value; ++it) {
      const int q = it * 256 + threadIdx.x;    // 2048 chunks: 256 rows x 8 chunks of a 128-byte line
      const int row = q >> 3, c8 = q & 7;
      const u32x4* src = W0;
      int64_t r;
      if (p.mode == 3) {
        int64_t slot = g_row0 + row;
        if (slot >= g_end) slot = g_end - 1;
        r = p.rows_of[slot];
      } else {
        if (p.mode == 0) r = (int64_t)t * 256 + row;
        else if (p.mode == 1) r = (int64_t)t * 256 + perm32(row);
        else {
          r = (int64_t)t * 128 + perm32(row & 127);
          if (row >= 128) src = W1;
        }
        if (r >= p.rows) r = p.rows - 1;
      }
      const u32x4 v = src[r * p.ld_chunks + (int64_t)sp * 8 + c8];
      const int s = 2 * sp + (c8 >> 2);
      const int pos = (c8 & 3) ^ ((row >> 2) & 3);
      dst[((int64_t)t * p.nsl + s) * 1024 + row * 4 + pos] = v;
    }
  };
  if (groups > 6) move(std::integral_constant<int, 8>{});
  else if (groups > 4) move(std::integral_constant<int, 6>{});
  else move(std::integral_constant<int, 4>{});
}

// ---- GEMM --------------------------------------------------------------------------------------
struct KArgs {
  const char* A;          // packed, tile-major
  const char* B;          // packed weight blocks; BROW: the weights as the caller stores them, row-major [N, K]
  const char* B1;         // BROW, gate/up: the linear branch
  void* C;                // EPI_STORE: row-major bf16 [M, ldc]; EPI_SWIGLU: packed A operand with K = N
  int64_t M, ldc;
  int N;                  // output columns
  int nsl;                // K / 32
  int m_tiles, n_tiles;   // dense; n_tiles: of the width the launch walks
  int half_width, row_groups;
  bool stream;            // the weights are far more than the caches hold
  // grouped mode (rows partitioned into per-expert segments, tile t = rows tile_row0[t] .. of expert
  // tile_expert[t]; A and a packed C are indexed by TILE, a row-major C by row)
  const int32_t* tile_expert; const int32_t* tile_row0; const int32_t* seg_end;
  int64_t b_expert_bytes;
  const float* row_scale;
  // dense batched mode: `experts` independent GEMMs of the same shape in one launch, tile ids expert-major;
  // expert e reads A + e a_expert_bytes (0: A shared), B + e b_expert_bytes, writes C + e c_expert_bytes
  int experts;
  int64_t a_expert_bytes, c_expert_bytes;
  // EPI_ROWSCALE_F32: rows with row_dest[r] >= 0 go, as bf16 and unscaled, to row row_dest[r] of direct_out
  const int32_t* row_dest;
  uint16_t* direct_out;
  const uint32_t* tile_order;   // grouped mode: a header, then entry bid = (M tile << 12) | N tile
};

// Round counters of the persistent workgroups, one per XCD (64 bytes apart); see round_sync in the kernel.
// They only ever grow, by a multiple of the XCD's workgroup count per launch; 64 bits wide, so they never wrap.
// Launches that overlap on one GPU share them: their workgroups may then wait for each other up to the
// bound, nothing else.  Workgroup b is taken to run on XCD b % 8 (how this part deals workgroups out); were
// that ever not so, the line-ups would group the wrong workgroups and cost time, never a result.
__device__ unsigned long long g_round_count[8 * 8];

// NG: accumulator tiles of a wavefront along N: 8, or 4 for tiles of half the width.  MG: along M: 8, or 6 or 4 for launches
// none of whose tiles has more than 192 or 128 rows (the rows beyond are neither fetched nor multiplied).
// STREAM: the weights' loads carry the non-temporal hint.
template <int EPI, bool GROUPED, bool BROW, int NG, int MG, bool STREAM>
__device__ __forceinline__ void gemm_body() {
  // (the kernel's arguments, through a pointer the compiler cannot see through: it would load what all bodies use before it
  // picks one, and hold it in scalar registers that the loops need; they start the kernel-argument segment, being the only
  // parameter: asserted at the kernel)
  typedef const __attribute__((address_space(4))) KArgs* args_t;
  args_t args = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  const __attribute__((address_space(4))) KArgs& p = *args;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int wm = wave_u >> 1, wn = wave_u & 1;
  const int nsl = p.nsl;
  // Grouped launches are sized for the largest possible tile map; the order says how many tiles there are: full-width ones first,
  // half-width ones after them.
  const uint32_t m_tiles = (uint32_t)p.m_tiles, n_tiles = (uint32_t)p.n_tiles;
  const uint32_t per_expert = m_tiles * n_tiles;
  const uint32_t nblk = GROUPED ? p.tile_order[NG == 8 ? TILE_ORDER_FULL : TILE_ORDER_HALF] : per_expert * (uint32_t)p.experts;
  const uint32_t order_at = TILE_ORDER_HEADER + (GROUPED && NG == 4 ? p.tile_order[TILE_ORDER_FULL] : 0u);
  const uint32_t G = gridDim.x;

  // Logical tile id -> (tm, tn).  Ids i, i + 8, ... belong to XCD i % 8 (the grid is a multiple of 8 or
  // a single round); every XCD gets a contiguous run of tiles, GROUP_M M-tiles deep.
  constexpr uint32_t GROUP_M = (EPI == EPI_SWIGLU ? GEMM_GROUP_M_SWIGLU : GEMM_GROUP_M_STORE) * NG / 8;
  // weight blocks of the tile's expert (BROW: the first of this wavefront's 64 or 32 weight rows; rows come in whole groups of
  // 64, a group beyond the last one re-reads that, its products are never stored)
  const int pitch = nsl * 64;
  const int brow_group = NG == 8 ? 32 * wave_u : 32 * (wave_u >> 1);
  const int brow_uni = NG == 8 ? 0 : 4 * (wave_u & 1) * pitch;
  auto b_tile = [&](int tm_, int tn_, int e_, int unit) {
    const char* b;
    if (BROW) {
      // a unit: 16 NG rows of either branch, or half of the tile's 32 NG; a wavefront brings 4 NG of them
      const int row = EPI == EPI_SWIGLU ? tn_ * (16 * NG) : tn_ * (32 * NG) + unit * (16 * NG);
      b = (EPI == EPI_SWIGLU && unit ? p.B1 : p.B) + (int64_t)min(row + brow_group, p.N - 32) * pitch + brow_uni;
    } else if (NG == 8) {
      b = p.B + ((size_t)tn_ * nsl) * SLICE + wave_u * 4096;
    } else {                                      // half a block: 128 rows, or 64 gate rows and the same 64 up rows
      b = p.B + ((size_t)(tn_ >> 1) * nsl) * SLICE +
          (EPI == EPI_SWIGLU ? (tn_ & 1) * 4096 + (wave_u >> 1) * 8192 + (wave_u & 1) * 2048 : (tn_ & 1) * 8192 + wave_u * 2048);
    }
    b += (int64_t)(GROUPED ? __builtin_amdgcn_readfirstlane(p.tile_expert[tm_]) : e_) * p.b_expert_bytes;
    return b;
  };
  // Dense: e = the GEMM of a batched launch the tile belongs to; each of them is dealt to the XCDs exactly as a
  // launch of its own would be when its tile count is a multiple of 8 and the launch takes several rounds, else the batch
  // is one flat run of tiles (in a single round that keeps an expert's operands on one XCD).
  auto decode = [&](uint32_t L, int& tm, int& tn, int& e) {
    const uint32_t xcd = L & 7, j = L >> 3;
    if (GROUPED) {
      // the order of the tiles was laid out by the caller (groups of M tiles aligned to experts, see write_order in skip.hip);
      // XCD x walks entries x per + min(x, rem) ... of it
      const uint32_t per = nblk >> 3, rem = nblk & 7;
      const uint32_t v = p.tile_order[order_at + xcd * per + (xcd < rem ? xcd : rem) + j];
      e = 0;
      tm = (int)(v >> 12);
      tn = (int)(v & 4095u);
    } else {
      uint32_t bid;
      if ((per_expert & 7) == 0 && nblk > G) {
        const uint32_t per8 = per_expert >> 3;
        const uint32_t eu = j / per8;
        e = (int)eu;
        bid = xcd * per8 + (j - eu * per8);
      } else {
        const uint32_t per = nblk >> 3, rem = nblk & 7;
        bid = xcd * per + (xcd < rem ? xcd : rem) + j;
        const uint32_t eu = bid / per_expert;
        e = (int)eu;
        bid -= eu * per_expert;
      }
      const uint32_t group_sz = GROUP_M * n_tiles;
      const uint32_t group = bid / group_sz;
      const uint32_t first_m = group * GROUP_M;
      const uint32_t gm = min(m_tiles - first_m, GROUP_M);
      const uint32_t in_group = bid - group * group_sz;
      tm = (int)(first_m + in_group % gm);
      tn = (int)(in_group / gm);
    }
    // (the divisions above went through vector registers)
    tm = __builtin_amdgcn_readfirstlane(tm);
    tn = __builtin_amdgcn_readfirstlane(tn);
    e = __builtin_amdgcn_readfirstlane(e);
  };

  // ---- loader state (all wave-uniform) ----------------------------------------------------------
  // A wavefront moves 4 KB of each operand block per slice: KB 4 w .. 4 w + 3.
  uint32_t L_ld = blockIdx.x;
  if (L_ld >= nblk) return;
  int tm_ld, tn_ld, e_ld;
  decode(L_ld, tm_ld, tn_ld, e_ld);
  const char* a_ld = p.A + (int64_t)e_ld * p.a_expert_bytes + ((size_t)tm_ld * nsl) * SLICE + wave_u * (MG * 512);
  const char* b_ld = b_tile(tm_ld, tn_ld, e_ld, 0);
  // BROW: from the tile's first unit to its second
  const int64_t b1_branch = p.B1 - p.B;
  int b1_rows = BROW && EPI != EPI_SWIGLU ? (int)(b_tile(tm_ld, tn_ld, e_ld, 1) - b_ld) : 0;
  int s_ld = 0;
  int st_ld = 0;                      // byte offset of the stage the next slice goes to
  bool ld_ok = true;
  const int lane_off = lane * 16;
  typedef __attribute__((address_space(3))) char lds_char;
  lds_char* const lds3 = (lds_char*)lds;
  // packed: per-lane global addresses of this wavefront's part of the next slice (kept in registers so that the
  // step that issues the loads has no address arithmetic to do first)
  const char* ga = a_ld + lane_off;
  const char* gb = b_ld + lane_off;
  // BROW: lane l brings position l % 8 of LDS row 8 j + l / 8 of a group of 32, j = 0 .. 3 the load: weight row
  // (l / 8) % 4 + 8 (l / 32) + 16 (j % 2) + 4 (j / 2), chunk (l % 8) ^ (4 (j % 2) + l / 16).
  const int brow_even = (8 * (lane >> 5) + ((lane >> 3) & 3)) * pitch + (((lane & 7) ^ (lane >> 4)) << 4);
  const int brow_odd = brow_even ^ 64;
  // BROW loads go through buffer descriptors: a scalar base, a 32-bit lane offset and a scalar offset, so that a step has no
  // vector additions to do for its addresses (with 64-bit vector addresses it had 8, and too few registers left to spread the
  // loads over the step).  On packed operands, one address register pair each, plain loads are 1 % faster.
  typedef __attribute__((address_space(3))) void* lds_t;
  typedef const __attribute__((address_space(1))) void* gptr_t;
#define MOEP_BUFFER_LOAD(base, lane_offset, offset, dst, imm, hint)                             \
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)(base), 0, -1, 0x00027000), \
      (lds_t)(lds3 + (dst)), 16, lane_offset, offset, imm, hint);
#define MOEP_LOAD_A(q)                                                                          \
  if constexpr (!BROW) __builtin_amdgcn_global_load_lds((gptr_t)ga, (lds_t)(lds3 + st_ld + wave_u * (MG * 512)), 16, (q) * 1024, 0); \
  else MOEP_BUFFER_LOAD(a_ld, lane_off, 0, st_ld + wave_u * (MG * 512), (q) * 1024, 0)
#define MOEP_LOAD_B(q, unit)                                                                    \
  if constexpr (!BROW) __builtin_amdgcn_global_load_lds((gptr_t)gb, (lds_t)(lds3 + RING + st_ld + wave_u * (NG * 512)), 16, (q) * 1024, STREAM ? 2 : 0); \
  else MOEP_BUFFER_LOAD(b_ld + ((unit) ? (EPI == EPI_SWIGLU ? b1_branch : (int64_t)b1_rows) : 0),  \
                        (q) & 1 ? brow_odd : brow_even, (16 * ((q) & 1) + 4 * ((q) >> 1)) * pitch, \
                        RING + st_ld + wave_u * (NG * 512) + (q) * 1024, 0, STREAM ? 2 : 0)
  // After a slice has been issued: next slice, next stage (branch-free, so that it can be scheduled into
  // the shadow of the MFMAs).  Past the end of the workgroup's stream the loader stays on its last slice:
  // the re-reads are in bounds and land in stages nobody reads again, every step issues the same loads and
  // the wait counts below hold to the end.
#define MOEP_ADVANCE_LOADER(unit)                                                               \
  {                                                                                             \
    a_ld += ld_ok ? SLICE : 0;                                                                  \
    if (!BROW) b_ld += ld_ok ? SLICE : 0;                                                       \
    else if (unit) b_ld += ld_ok ? 128 : 0;                                                     \
    s_ld += ld_ok ? 1 : 0;                                                                      \
    st_ld = st_ld + SLICE == RING ? 0 : st_ld + SLICE;                                          \
    if (!BROW) { ga = a_ld + lane_off; gb = b_ld + lane_off; }                                  \
  }
  // The workgroups of an XCD start every SYNC_EVERY-th round of tiles together: they share operand panels through the
  // XCD's L2 only while they walk K within a few steps of each other, and left alone they settle, from
  // one build of this file to the next, either there or in a state where every panel is fetched about three
  // times over (L2 hit rate 0.45 instead of 0.80, 7 % slower).  Arrivals are counted in a counter that only
  // grows.  A workgroup has `rounds` tiles or one fewer, and there is a line-up after every SYNC_EVERY tiles except the last
  // round's: every workgroup arrives at every one of them, once (one that has no further tile does not wait), so the count stays
  // a multiple of the XCD's workgroup count from line-up to line-up and from launch to launch.  (When workgroups without a
  // further tile arrived for the line-ups to come as well, those that had one waited for a count that the launch could not
  // reach, up to the bound: gate/up, K = 512, 4.25 rounds took 110 us where 5 take 80; 78 now.)  The wait is bounded (SYNC_POLLS polls about a
  // thousand cycles apart); a workgroup that ran into the bound goes on alone and polls no more in this launch.  Only the
  // timing depends on any of this, never a result.
  const uint32_t rounds = (nblk + G - 1) / G;
  const bool sync_on = nblk > G && (G & 7) == 0 && (G >> 3) < 65536u;
  bool poll_ok = true;
  uint32_t switches = 0;
  auto round_sync = [&](bool wait) {
    int w_ = wave_u;                          // (opaque: the comparison is then made here, from a scalar register,
    asm volatile("" : "+s"(w_));              // instead of being kept as a 0/1 value in a vector register across the K loop)
    if (w_ != 0) return;
    unsigned long long* c = &g_round_count[(blockIdx.x & 7) * 8];
    unsigned long long old_v = 0;
    if (lane == 0)
      old_v = __hip_atomic_fetch_add(c, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!wait || !poll_ok) return;
    // Everyone has arrived when the count reaches the next multiple of n above the value this arrival saw.
    // (wave-uniform 32-bit arithmetic: old mod n from the two halves of the 64-bit count, n < 2^16)
    const uint32_t n = G >> 3;
    const uint32_t old_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)old_v);
    const uint32_t old_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(old_v >> 32));
    const uint32_t two32_mod_n = (0xffffffffu % n + 1u) % n;
    const uint32_t old_mod_n = ((old_hi % n) * two32_mod_n + old_lo % n) % n;
    const uint32_t target_lo = old_lo - old_mod_n + n;          // low word of the target; the count moves by far
    int polls = 0;                                              // less than 2^31 while this workgroup waits
    for (;;) {
      uint32_t now_v = 0;
      if (lane == 0) now_v = (uint32_t)__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t now = (uint32_t)__builtin_amdgcn_readfirstlane((int)now_v);
      if ((int32_t)(now - target_lo) >= 0) break;
      if (++polls >= SYNC_POLLS) { poll_ok = false; break; }
      __builtin_amdgcn_s_sleep(16);
    }
  };
  // ... and, between runs of steps, the next tile of this workgroup
#define MOEP_NEXT_LOAD_TILE()                                                                   \
  if (s_ld == nsl) {                                                                            \
    s_ld = 0;                                                                                   \
    L_ld += G;                                                                                  \
    ++switches;                                                                                 \
    if (sync_on && switches % SYNC_EVERY == 0 && switches < rounds) {                           \
      round_sync(L_ld < nblk);                                                                  \
      __builtin_amdgcn_s_barrier();                                                             \
    }                                                                                           \
    if (L_ld < nblk) {                                                                          \
      decode(L_ld, tm_ld, tn_ld, e_ld);                                                         \
      a_ld = p.A + (int64_t)e_ld * p.a_expert_bytes + ((size_t)tm_ld * nsl) * SLICE + wave_u * (MG * 512); \
      b_ld = b_tile(tm_ld, tn_ld, e_ld, 0);                                                     \
      if (BROW && EPI != EPI_SWIGLU) b1_rows = (int)(b_tile(tm_ld, tn_ld, e_ld, 1) - b_ld);      \
    } else {                                                                                    \
      ld_ok = false;                                                                            \
      a_ld -= SLICE;                                                                            \
      b_ld -= BROW ? 128 : SLICE;                                                               \
    }                                                                                           \
    if (!BROW) { ga = a_ld + lane_off; gb = b_ld + lane_off; }                                  \
  }

  // ---- fragment addresses -------------------------------------------------------------------------
  // MFMA 16x16x32: lane l supplies row (l & 15) and k-values 8 (l >> 4) .. + 7 of both operands, i.e.
  // chunk (l >> 4) of the row, found at the position that the layout gives it; tile rows are multiples of 16
  // apart, so the permutation depends on the lane only and every fragment is base + constant.
  const int frow = lane & 15, fk = lane >> 4;
  const int fpos = (fk ^ ((frow >> 2) & 3)) << 4;
  const int a_fb = (wm * (MG * 16) + frow) * 64 + fpos;
  // BROW: rows of 128 bytes, two slices wide, chunk c of row r at position c ^ ((r >> 1) & 7); a slice's fragments lie in the
  // pair's two units (gate rows in one, up rows in the other; plain: wavefront column wn's rows are unit wn).
  const int b_fb = RING + (BROW ? ((EPI == EPI_SWIGLU ? wn * (NG * 8) : 0) + frow) * 128 + ((fk ^ ((frow >> 1) & 7)) << 4)
                                : ((EPI == EPI_SWIGLU ? wn * (NG * 8) : wn * (NG * 16)) + frow) * 64 + fpos);
  int st_rd = 0;                      // byte offset of the stage the next fragment read takes
  int ra = a_fb;                      // the same, added to the lane's fragment offsets
  int rb = b_fb, rb1 = b_fb;          // BROW, gate/up: rb1 = the up rows' unit
  int su = 0;                         // BROW: byte offset of the first unit of the pair of slices to be read next
#define MOEP_NEXT_UNIT(u) ((u) + SLICE == RING ? 0 : (u) + SLICE)
  // fragment addresses of the second (half 1) or first slice of the pair at `su`; after the second one the next pair's turn
#define MOEP_B_ADDRESS(half)                                                                    \
  if (BROW) {                                                                                   \
    const int su1 = MOEP_NEXT_UNIT(su);                                                         \
    rb = (b_fb ^ ((half) * 64)) + (EPI == EPI_SWIGLU || !wn ? su : su1);                        \
    rb1 = (b_fb ^ ((half) * 64)) + su1;                                                         \
    if (half) su = MOEP_NEXT_UNIT(su1);                                                         \
  } else {                                                                                      \
    rb = b_fb + st_rd;                                                                          \
  }

  f32x4 acc[MG][NG];
#define MOEP_ZERO_ACC()                                                                         \
  _Pragma("unroll") for (int i = 0; i < MG; ++i)                                                \
    _Pragma("unroll") for (int j = 0; j < NG; ++j)                                              \
      _Pragma("unroll") for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
  bf16x8 fa[2][MG], fb[2][NG];
  // B tile j of a wavefront: SwiGLU: gate tiles 0 .. NG/2 - 1 and up tiles (NG 16 rows further) of the same
  // 8 NG columns; otherwise NG consecutive 16-row tiles.
#define MOEP_RB(slot, j)                                                                        \
  fb[slot][j] = *(const bf16x8*)(lds + (!BROW ? rb + (EPI == EPI_SWIGLU ? ((j) / (NG / 2)) * (NG * 1024) + ((j) % (NG / 2)) * 1024 : (j) * 1024) \
      : EPI == EPI_SWIGLU ? ((j) < NG / 2 ? rb : rb1) + ((j) % (NG / 2)) * 2048 : rb + (j) * 2048));
#define MOEP_RA(slot, i) fa[slot][i] = *(const bf16x8*)(lds + ra + (i) * 1024);
  // (B fragments visited back and forth, so that only one operand changes from one MFMA to the next: 0.6 % faster)
#define MOEP_MFMA(slot)                                                                         \
  _Pragma("unroll") for (int i = 0; i < MG; ++i)                                                \
    _Pragma("unroll") for (int jj = 0; jj < NG; ++jj) {                                         \
      const int j = (i & 1) ? NG - 1 - jj : jj;                                                 \
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[slot][j], fa[slot][i], acc[i][j], 0, 0, 0); }
  // Source order = wanted issue order (a direct load writes LDS, so the compiler keeps it ordered with
  // the fragment reads around it): two fragment reads, one direct load, over and over, spread over
  // the step's MFMAs by the scheduling groups below.
// (BROW: the weights' loads first, which the waits below count on; the unit is the one of the step that issues them, slot ^ 1)
#define MOEP_LOADN(n, unit)                                                                     \
  {                                                                                             \
    constexpr int nb_ = NG / 2, na_ = MG / 2;                                                   \
    if constexpr ((n) < na_ + nb_) {                                                            \
      if constexpr (BROW) { if constexpr ((n) < nb_) { MOEP_LOAD_B(n, unit) } else { MOEP_LOAD_A((n) - nb_) } } \
      else { if constexpr ((n) < na_) { MOEP_LOAD_A(n) } else { MOEP_LOAD_B((n) - na_, unit) } } \
    }                                                                                           \
  }
#define MOEP_READN(slot, n)                                                                     \
  { if constexpr ((n) < NG) { MOEP_RB(slot, n) } else if constexpr ((n) < NG + MG) { MOEP_RA(slot, (n) - NG) } }
#define MOEP_READS_LOADS(slot, unit)                                                            \
    MOEP_READN(slot, 0) MOEP_READN(slot, 1) MOEP_LOADN(0, unit) MOEP_READN(slot, 2) MOEP_READN(slot, 3) MOEP_LOADN(1, unit) \
    MOEP_READN(slot, 4) MOEP_READN(slot, 5) MOEP_LOADN(2, unit) MOEP_READN(slot, 6) MOEP_READN(slot, 7) MOEP_LOADN(3, unit) \
    MOEP_READN(slot, 8) MOEP_READN(slot, 9) MOEP_LOADN(4, unit) MOEP_READN(slot, 10) MOEP_READN(slot, 11) MOEP_LOADN(5, unit) \
    MOEP_READN(slot, 12) MOEP_READN(slot, 13) MOEP_LOADN(6, unit) MOEP_READN(slot, 14) MOEP_READN(slot, 15) MOEP_LOADN(7, unit)
#define MOEP_READS(slot)                                                                        \
  _Pragma("unroll") for (int j_ = 0; j_ < NG; ++j_) { MOEP_RB(slot, j_) }                       \
  _Pragma("unroll") for (int i_ = 0; i_ < MG; ++i_) { MOEP_RA(slot, i_) }
  // Two MFMAs, a fragment read, two MFMAs, a fragment read, two MFMAs, a direct load: never more than one
  // memory instruction between two MFMAs (1 % faster than 3 + read + 3 + read + load).  Smaller tiles have fewer MFMAs for them.
#define MOEP_SCHED()                                                                            \
  _Pragma("unroll") for (int q_ = 0; q_ < (MG + NG) / 2; ++q_) {                                \
    constexpr int per_ = 2 * MG * NG / (MG + NG);                                               \
    __builtin_amdgcn_sched_group_barrier(0x008, per_ > 3 ? 2 : 1, 0);                           \
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                          \
    __builtin_amdgcn_sched_group_barrier(0x008, per_ > 4 ? 2 : 1, 0);                           \
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                          \
    __builtin_amdgcn_sched_group_barrier(0x008, per_ > 5 ? 2 : 1, 0);                           \
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                          \
  }
  // s_waitcnt immediates: vmcnt in bits 3:0 and 15:14, lgkmcnt in bits 11:8 (0 here), expcnt 6:4 left at 7.
  // Loads complete in issue order, so "at most STEP_LOADS outstanding" means that everything but the slice issued in
  // this step has landed, in particular the two slices whose fragments are read before the next barrier
  // (stores of an epilogue only add to the count).
  // BROW: a pair's second unit is issued one step before the first slice that needs it is read, so there is a barrier after
  // every step.  Before an odd step all but the loads from the newest unit's slice of A on have to have landed, before an even
  // step all but those of the two newest steps.  (The unit that an odd step's loads overwrite was read in the step before:
  // those reads are back, lgkmcnt 0, before the barrier.)
  constexpr int STEP_LOADS = MG / 2 + NG / 2;
  constexpr auto wait_for = [](int vm) { return 0x0070 | (vm & 15) | ((vm >> 4) << 14); };
  constexpr int W_MAIN = wait_for(BROW ? 2 * STEP_LOADS : STEP_LOADS), W_ODD = wait_for(STEP_LOADS + MG / 2);
  // One step: multiply the slice whose fragments are in `slot`; meanwhile fetch the slice NS - 1 ahead and
  // read the next slice's fragments into the other slot.  The barrier at the end of every second step tells
  // every wavefront that the next two slices have landed for all of them and that all of them have read
  // the fragments of the two stages that the next two steps' loads overwrite.
#define MOEP_STEP(slot, BAR)                                                                    \
  {                                                                                             \
    MOEP_READS_LOADS((slot) ^ 1, slot)                                                          \
    MOEP_MFMA(slot)                                                                             \
    MOEP_SCHED()                                                                                \
    MOEP_ADVANCE_LOADER(slot)                                                                   \
    st_rd = st_rd + SLICE == RING ? 0 : st_rd + SLICE;                                          \
    ra = a_fb + st_rd;                                                                          \
    MOEP_B_ADDRESS(slot)                                                                        \
    __builtin_amdgcn_sched_barrier(0);                                                          \
    if (BAR || BROW) {                                                                          \
      __builtin_amdgcn_s_waitcnt(BAR ? W_MAIN : W_ODD);                                         \
      __builtin_amdgcn_s_barrier();                                                             \
    }                                                                                           \
    __builtin_amdgcn_sched_barrier(0);                                                          \
  }

  // ---- prologue: the first NS - 1 slices of this workgroup's stream -----------------------------------
#pragma unroll 1
  for (int n = 0; n < NS - 1; n += 2) {
#define MOEP_LOADS(unit)                                                                        \
    MOEP_LOADN(0, unit) MOEP_LOADN(1, unit) MOEP_LOADN(2, unit) MOEP_LOADN(3, unit)             \
    MOEP_LOADN(4, unit) MOEP_LOADN(5, unit) MOEP_LOADN(6, unit) MOEP_LOADN(7, unit)             \
    MOEP_ADVANCE_LOADER(unit)
    MOEP_LOADS(0)
    MOEP_LOADS(1)
    MOEP_NEXT_LOAD_TILE()
  }
  __builtin_amdgcn_s_waitcnt(0x0070);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  MOEP_B_ADDRESS(0)
  MOEP_READS(0)
  st_rd = SLICE;
  ra = a_fb + st_rd;
  MOEP_B_ADDRESS(1)
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): stage 0 is overwritten by the second step's loads, and
  __builtin_amdgcn_s_barrier();         // no barrier separates it from these reads otherwise
  __builtin_amdgcn_sched_barrier(0);

  uint32_t L_mm = blockIdx.x;
  int tm, tn, e_mm;
  decode(L_mm, tm, tn, e_mm);
  for (;;) {
    MOEP_ZERO_ACC()
    // The loader is NS - 1 slices ahead and changes tile between two runs of steps, never inside one.  K / 32
    // and NS - 1 are even, so every run is a whole number of step pairs.
    for (int left = nsl; left > 0;) {
      const int run = min(left, nsl - s_ld);
#pragma unroll 1
      for (int s_mm = 0; s_mm < run; s_mm += 2) {
        MOEP_STEP(0, false)
        MOEP_STEP(1, true)
      }
      left -= run;
      MOEP_NEXT_LOAD_TILE()
    }

    // ---- epilogue of tile (tm, tn) ------------------------------------------------------------------
    // Register v of lane l of accumulator tile (i, j) holds output row 16 i + (l % 16) of the wavefront's
    // 128 rows and fragment row f = 4 (l / 16) + v of weight tile j; with the row permutation of the weight
    // blocks, tiles 2 P and 2 P + 1 together give the lane the 8 consecutive columns 32 P + 8 (l / 16) .. + 7.
    // The lane id is recomputed here, in a form the compiler cannot move: anything derived from a value that
    // lives across the K loop is hoisted above it and held (or spilled) there, and the loop has no register to spare.
    int lane_e;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane_e));
    const int q8 = 8 * (lane_e >> 4);
    int64_t row0 = (int64_t)tm * 256, row_end = p.M;
    if (GROUPED) {
      row0 = p.tile_row0[tm];
      row_end = p.seg_end[p.tile_expert[tm]];
    }
    char* const c_base = (char*)p.C + (GROUPED ? (int64_t)0 : (int64_t)e_mm * p.c_expert_bytes);
    // EPI_ROWSCALE_F32: scales and destinations of the wavefront's rows, 64 to a register, all fetched before the first is used
    // (row group by row group they were 16 round trips to memory, one after the other: E 16, H 2048, F 5632, top-4, 1001 tokens, this
    // launch 151 -> 147 us; Mixtral shape, 32768 tokens, the forward 13190 -> 13110)
    constexpr int ROW_REGS = EPI == EPI_ROWSCALE_F32 ? (MG + 3) / 4 : 1;
    float scales[ROW_REGS];
    int dests[ROW_REGS];
    if (EPI == EPI_ROWSCALE_F32) {
#pragma unroll
      for (int q = 0; q < ROW_REGS; ++q) {
        int64_t r = row0 + wm * (MG * 16) + 64 * q + lane_e;
        if (r >= row_end) r = row_end - 1;
        scales[q] = p.row_scale[r];
        dests[q] = p.row_dest ? p.row_dest[r] : -1;
      }
    }
#pragma unroll
    for (int i = 0; i < MG; ++i) {
      const int prow = wm * (MG * 16) + i * 16 + (lane_e & 15);          // row inside the tile
      const int64_t r = row0 + prow;
      float sc = 0.f;
      int dest = -1;                                             // >= 0: this row is a token's only slot
      if (EPI == EPI_ROWSCALE_F32) {                             // (by all lanes: they fetch from each other)
        const int from = 4 * ((i & 3) * 16 + (lane_e & 15));
        sc = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(scales[i / 4 < ROW_REGS ? i / 4 : 0])));
        dest = __builtin_amdgcn_ds_bpermute(from, dests[i / 4 < ROW_REGS ? i / 4 : 0]);
      }
      if (r >= row_end) continue;
      if (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int P = 0; P < NG / 4; ++P) {
        const int n = tn * (NG * 16) + wn * (NG * 8) + 32 * P + q8;
        if (n < p.N) {
          bf16x2 o[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            f32x2 h;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
              const int b = 2 * P + (c >> 1), v = 2 * (c & 1) + d;
              const float g = acc[i][b][v], u = acc[i][NG / 2 + b][v];
              h[d] = g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
            }
            o[c] = __builtin_convertvector(h, bf16x2);
          }
          // packed A operand with K = N: slice n / 32, chunk (l / 16) of row prow
          char* dst = c_base + ((size_t)tm * (p.N >> 5) + (n >> 5)) * SLICE + prow * 64 +
                      (((lane_e >> 4) ^ ((prow >> 2) & 3)) << 4);
          *(u32x4*)dst = __builtin_bit_cast(u32x4, o);
        }
        }
      } else {
#pragma unroll
        for (int P = 0; P < NG / 2; ++P) {
          const int n = tn * (NG * 32) + wn * (NG * 16) + 32 * P + q8;
          if (n >= p.N) continue;
          if (EPI == EPI_STORE || (EPI == EPI_ROWSCALE_F32 && dest >= 0)) {
            bf16x2 o[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const f32x2 h = {acc[i][2 * P + (c >> 1)][2 * (c & 1)], acc[i][2 * P + (c >> 1)][2 * (c & 1) + 1]};
              o[c] = __builtin_convertvector(h, bf16x2);
            }
            uint16_t* const row = EPI == EPI_STORE ? (uint16_t*)c_base + r * p.ldc : p.direct_out + (int64_t)dest * p.ldc;
            *(u32x4*)(row + n) = __builtin_bit_cast(u32x4, o);
          } else {                                               // EPI_ROWSCALE_F32
            float* dst = (float*)c_base + r * p.ldc + n;
            *(f32x4*)dst = sc * acc[i][2 * P];
            *(f32x4*)(dst + 4) = sc * acc[i][2 * P + 1];
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    L_mm += G;
    if (L_mm >= nblk) break;   // (the loads still in flight are re-reads; the wavefront ends when they are back)
    decode(L_mm, tm, tn, e_mm);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);   // the re-reads still in flight target this workgroup's LDS
#undef MOEP_BUFFER_LOAD
#undef MOEP_LOAD_A
#undef MOEP_LOAD_B
#undef MOEP_LOADN
#undef MOEP_READN
#undef MOEP_LOADS
#undef MOEP_NEXT_UNIT
#undef MOEP_B_ADDRESS
#undef MOEP_ADVANCE_LOADER
#undef MOEP_NEXT_LOAD_TILE
#undef MOEP_ZERO_ACC
#undef MOEP_RB
#undef MOEP_RA
#undef MOEP_MFMA
#undef MOEP_READS_LOADS
#undef MOEP_READS
#undef MOEP_SCHED
#undef MOEP_STEP
}

// The body is picked by the launch's row groups and tile width.  Row groups: of a launch whose tallest tile has up to 128 or 192
// rows only those are fetched and multiplied.  By themselves, without the cut into shorter tiles (tile_plan.h), us per
// skipping forward, Mixtral shape, median of three processes each way: T = 300 (75 rows per expert) 712 -> 598, 450 719 -> 600,
// 777 737 -> 659; dense pass of 128 tokens 700 -> 581, of 192 707 -> 631.  They are bodies of their own: with one
// accumulator array and a loop per height the register allocator spilled some 400 registers around the loops.
// A launch of tiles of up to 128 rows reads every expert's weights once (an expert has one tile): where they are far more than
// the caches hold, they come with the non-temporal hint.  Without / with, us per call, no token skipped: Mixtral shape, T = 200
// 570 / 552 (packed 576 / 537), 400 586 / 577 (588 / 565); E 16, H 2048, F 5632, T = 300 257 / 249; dense, 64 tokens, Mixtral shape
// 557 / 537.  Taller tiles gain nothing (T = 777 720 / 718).
// A launch with so few tiles that compute units would stand idle walks tiles of half the width instead, 256 x 128
// accumulator columns (64 outputs in SwiGLU mode), bits unchanged.  Half-width tiles cost well over half the time of full
// ones (the same rows of A per step), so they only pay while they still fit one round (half_width_pays).  Grouped launches
// learn from the tile order's header which it is: only the device knows how many tiles the routing made.
// Down projection 4096 x 14336, 8 experts of about 150 rows: 128 tiles 360 us, 256 of half the width 281 us.
template <int EPI, bool GROUPED, bool BROW>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_packed_kernel(KArgs p) {
  const bool full = GROUPED ? p.tile_order[TILE_ORDER_FULL] != 0 : p.half_width == 0;
  const bool half = GROUPED ? p.tile_order[TILE_ORDER_HALF] != 0 : p.half_width != 0;
  const uint32_t mg = GROUPED ? p.tile_order[TILE_ORDER_ROW_GROUPS] : (uint32_t)p.row_groups;
#define MOEP_BODY(NG)                                                                           \
  if (mg > 6) gemm_body<EPI, GROUPED, BROW, NG, 8, false>();                                   \
  else if (mg > 4) gemm_body<EPI, GROUPED, BROW, NG, 6, false>();                              \
  else if (p.stream) gemm_body<EPI, GROUPED, BROW, NG, 4, true>();                             \
  else gemm_body<EPI, GROUPED, BROW, NG, 4, false>();
  if (full) { MOEP_BODY(8) }
  if (GROUPED && full && half) __builtin_amdgcn_s_barrier();   // (the ring begins anew: all have read what it held)
  if (half) { MOEP_BODY(4) }
#undef MOEP_BODY
}
static_assert(std::is_same<decltype(gemm_packed_kernel<EPI_STORE, false, false>), void(KArgs)>::value &&
              std::is_trivially_copyable<KArgs>::value, "gemm_body finds KArgs at the start of the kernel-argument segment");

// Per-device launch state, filled on a device's first launch under a mutex (first calls from several host threads are
// safe): the compute-unit count, and whether the dynamic LDS limits have been raised.  They are raised for EVERY expert
// GEMM at once, so that after one call at any size a call at any other only launches (and can be captured).
constexpr int kMaxDevices = 64;
struct DeviceState {
  int compute_units = 0;
  bool ready = false;
};
std::mutex g_dev_mu;
DeviceState g_dev[kMaxDevices];

template <int EPI, bool GROUPED, bool BROW>
int allow_lds() {
  MOEP_HIP(hipFuncSetAttribute((const void*)gemm_packed_kernel<EPI, GROUPED, BROW>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES));
  return MOEP_OK;
}

template <int EPI, bool GROUPED, bool BROW>
int launch(const KArgs& k, hipStream_t s) {
  int cus = 0;
  if (int st = gemm_device_ready(&cus)) return st;
  const int64_t nblk = (int64_t)k.m_tiles * k.n_tiles * k.experts;
  int grid = cus & ~7;                        // one persistent workgroup per compute unit, a multiple of 8
  if (grid < 8) grid = 8;
  if (nblk < grid) grid = (int)nblk;          // a single round: any size
  hipLaunchKernelGGL((gemm_packed_kernel<EPI, GROUPED, BROW>), dim3(grid), dim3(THREADS), LDS_BYTES, s, k);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

int launch_pack(PackArgs p, int64_t tiles, int K, int experts, hipStream_t s, const char* name) {
  if (K <= 0 || K % 64) return fail(MOEP_EUNSUPPORTED, "%s: K=%d must be a positive multiple of 64", name, K);
  if (tiles <= 0 || experts <= 0) return MOEP_OK;
  if (((uintptr_t)p.W0 | (uintptr_t)p.W1 | (uintptr_t)p.dst) & 15)
    return fail(MOEP_EUNSUPPORTED, "%s: operands must be 16-byte aligned", name);
  if (tiles >= ((int64_t)1 << 31) || K / 64 > 65535 || experts > 65535) return fail(MOEP_EUNSUPPORTED, "%s: too large", name);
  p.nsl = K / 32;
  Timed t(name, s);
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)tiles, K / 64, experts), dim3(256), 0, s, p);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace

int gemm_device_ready(int* compute_units) {
  int dev = 0;
  MOEP_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(MOEP_EUNSUPPORTED, "device ordinal %d beyond %d", dev, kMaxDevices - 1);
  std::lock_guard<std::mutex> lk(g_dev_mu);
  DeviceState& d = g_dev[dev];
  if (!d.ready) {
    int v = 0;
    MOEP_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
    d.compute_units = v > 0 ? v : 256;
    for (auto allow : {allow_lds<EPI_STORE, false, false>, allow_lds<EPI_STORE, false, true>, allow_lds<EPI_STORE, true, false>,
                       allow_lds<EPI_STORE, true, true>, allow_lds<EPI_SWIGLU, false, false>, allow_lds<EPI_SWIGLU, false, true>,
                       allow_lds<EPI_SWIGLU, true, false>, allow_lds<EPI_SWIGLU, true, true>,
                       allow_lds<EPI_ROWSCALE_F32, true, false>, allow_lds<EPI_ROWSCALE_F32, true, true>})
      if (int st = allow()) return st;
    d.ready = true;
  }
  if (compute_units) *compute_units = d.compute_units;
  return MOEP_OK;
}

size_t packed_a_bytes(int64_t rows, int K) {
  return (size_t)ceil_div(rows, 256) * 256 * (size_t)K * 2;
}

size_t packed_b_bytes(int N, int K, bool gate_up_pair) {
  return (size_t)ceil_div(N, gate_up_pair ? 128 : 256) * 256 * (size_t)K * 2;
}

int launch_pack_a_bf16(const void* X, int64_t ld, int64_t rows, int K, void* dst, hipStream_t s, const char* name) {
  if (ld % 8) return fail(MOEP_EUNSUPPORTED, "%s: leading dimension must be a multiple of 8", name);
  PackArgs p = {};
  p.W0 = (const u32x4*)X; p.dst = (u32x4*)dst; p.ld_chunks = ld / 8; p.rows = rows; p.mode = 0;
  return launch_pack(p, ceil_div(rows, 256), K, 1, s, name);
}

int launch_pack_a_gathered_bf16(const void* X, int64_t ld, const int32_t* rows_of, const int32_t* tile_expert,
                                const int32_t* tile_row0, const int32_t* seg_end, const int32_t* tiles_in_use,
                                const uint32_t* tile_order, int64_t max_tiles, int K, void* dst, hipStream_t s, const char* name) {
  if (ld % 8) return fail(MOEP_EUNSUPPORTED, "%s: leading dimension must be a multiple of 8", name);
  PackArgs p = {};
  p.W0 = (const u32x4*)X; p.dst = (u32x4*)dst; p.ld_chunks = ld / 8; p.mode = 3;
  p.rows_of = rows_of; p.tile_expert = tile_expert; p.tile_row0 = tile_row0; p.seg_end = seg_end;
  p.tiles_in_use = tiles_in_use; p.tile_order = tile_order;
  return launch_pack(p, max_tiles, K, 1, s, name);
}

int launch_pack_b_bf16(const void* W0, const void* W1, int N, int K, int experts, void* dst, hipStream_t s,
                       const char* name) {
  PackArgs p = {};
  p.W0 = (const u32x4*)W0; p.W1 = (const u32x4*)W1; p.dst = (u32x4*)dst;
  p.ld_chunks = K / 8; p.rows = N; p.mode = W1 ? 2 : 1;
  p.src_expert_chunks = (int64_t)N * (K / 8);
  p.dst_expert_chunks = (int64_t)(packed_b_bytes(N, K, W1 != nullptr) / 16);
  return launch_pack(p, ceil_div(N, W1 ? 128 : 256), K, experts, s, name);
}

int launch_gemm_bf16_packed(const PackedGemmArgs& g, hipStream_t s, const char* name) {
  if (g.K <= 0 || g.K % 64) return fail(MOEP_EUNSUPPORTED, "%s: K=%d must be a positive multiple of 64", name, g.K);
  if (g.N <= 0 || g.N % 32) return fail(MOEP_EUNSUPPORTED, "%s: N=%d must be a positive multiple of 32", name, g.N);
  if (g.M <= 0) return MOEP_OK;
  if (((uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C) & 15)
    return fail(MOEP_EUNSUPPORTED, "%s: operands must be 16-byte aligned", name);
  if (g.epilogue != EPI_SWIGLU && (g.ldc % 8 || g.ldc < g.N)) return fail(MOEP_EINVAL, "%s: bad leading dimension", name);
  const bool grouped = g.tile_expert != nullptr;
  if (grouped && (!g.tile_row0 || !g.seg_end || !g.tile_order || g.max_m_tiles <= 0))
    return fail(MOEP_EINVAL, "%s: incomplete tile map", name);
  if (g.epilogue == EPI_ROWSCALE_F32 && !g.row_scale) return fail(MOEP_EINVAL, "%s: row_scale is NULL", name);
  KArgs k = {};
  k.A = (const char*)g.A; k.B = (const char*)g.B; k.C = g.C;
  k.M = g.M; k.ldc = g.ldc; k.N = g.N; k.nsl = g.K / 32;
  k.tile_expert = g.tile_expert; k.tile_row0 = g.tile_row0; k.seg_end = g.seg_end;
  if (g.b_row_major) {
    if (g.N % 64 || ((uintptr_t)g.B1 & 15) || (g.epilogue == EPI_SWIGLU && !g.B1))
      return fail(MOEP_EUNSUPPORTED, "%s: row-major weights need N=%d to be a multiple of 64 and 16-byte alignment", name, g.N);
    k.B1 = (const char*)g.B1;
    k.b_expert_bytes = (int64_t)g.N * g.K * 2;
  } else {
    k.b_expert_bytes = (int64_t)packed_b_bytes(g.N, g.K, g.epilogue == EPI_SWIGLU);
  }
  k.row_scale = g.row_scale;
  if (g.experts < 1 || (grouped && g.experts != 1)) return fail(MOEP_EINVAL, "%s: bad batch count %d", name, g.experts);
  k.experts = g.experts; k.a_expert_bytes = g.a_expert_bytes; k.c_expert_bytes = g.c_expert_bytes;
  if (g.row_dest && (g.epilogue != EPI_ROWSCALE_F32 || !g.direct_out || ((uintptr_t)g.direct_out & 15)))
    return fail(MOEP_EINVAL, "%s: row_dest needs the row-scaled epilogue and a 16-byte aligned direct_out", name);
  k.row_dest = g.row_dest; k.direct_out = (uint16_t*)g.direct_out;
  k.tile_order = grouped ? g.tile_order : nullptr;
  if ((g.a_expert_bytes | g.c_expert_bytes) & 15) return fail(MOEP_EUNSUPPORTED, "%s: per-expert strides must be multiples of 16 bytes", name);
  const int64_t m_tiles = grouped ? g.max_m_tiles : ceil_div(g.M, 256);
  // (grouped: tiles for the larger possible grid; the order's header tells the kernel which width to walk)
  const int64_t n_full = ceil_div(g.N, gemm_tile_columns(g.epilogue == EPI_SWIGLU, false));
  const int64_t n_half = ceil_div(g.N, gemm_tile_columns(g.epilogue == EPI_SWIGLU, true));
  const bool half = !grouped && half_width_pays(m_tiles * n_full * g.experts);
  const int64_t n_tiles = grouped || half ? n_half : n_full;
  if (m_tiles * n_tiles * g.experts >= ((int64_t)1 << 31)) return fail(MOEP_EUNSUPPORTED, "%s: too many tiles", name);
  k.m_tiles = (int)m_tiles; k.n_tiles = (int)n_tiles; k.half_width = half ? 1 : 0;
  k.row_groups = gemm_row_groups(g.M);
  k.stream = grouped ? g.stream : streams_weights(g.N, g.K, g.epilogue == EPI_SWIGLU, g.experts);
  Timed t(name, s);
#define MOEP_GEMM_CASE(EPI, GROUPED) \
  return g.b_row_major ? launch<EPI, GROUPED, true>(k, s) : launch<EPI, GROUPED, false>(k, s)
  if (grouped) {
    switch (g.epilogue) {
      case EPI_STORE: MOEP_GEMM_CASE(EPI_STORE, true);
      case EPI_SWIGLU: MOEP_GEMM_CASE(EPI_SWIGLU, true);
      case EPI_ROWSCALE_F32: MOEP_GEMM_CASE(EPI_ROWSCALE_F32, true);
    }
  } else {
    switch (g.epilogue) {
      case EPI_STORE: MOEP_GEMM_CASE(EPI_STORE, false);
      case EPI_SWIGLU: MOEP_GEMM_CASE(EPI_SWIGLU, false);
    }
  }
#undef MOEP_GEMM_CASE
  return fail(MOEP_EINVAL, "%s: unsupported epilogue %d", name, g.epilogue);
}

}  // namespace moep
