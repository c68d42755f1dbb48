// Router logits l[t,e] = sum_h x[t,h] Wgate[e,h] (Sec. 3.1), fp32 result.
//
// Bandwidth-bound: x is read once, Wgate (E x H) stays in L1/L2.  bf16 goes through
// router_mfma_kernel below; fp32 storage (and bf16 with H not a multiple of 32) through this kernel: a wavefront takes four
// tokens at a time; lane l owns the h-chunks l, l + 64, ... of every row (16 bytes each), keeps
// 4 x E partial sums, which are added across the lanes by halving (below).  The summation
// order for a token depends on nothing but H, so the same token gives the same bits in any batch
// -- moe_expert_outputs and moe_forward_skip rely on that.
#include "common.h"
#include "router_few.h"

namespace moep {
namespace {

constexpr int TOK = 4;

template <bool BF16>
struct Chunk;                      // one 16-byte load and its fp32 expansion
template <>
struct Chunk<true> {
  static constexpr int N = 8;
  __device__ static void load(const void* row, int chunk, float (&v)[8]) {
    const uint4 u = ((const uint4*)row)[chunk];
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __builtin_bit_cast(float, w[i] << 16);
      v[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xffff0000u);
    }
  }
};
template <>
struct Chunk<false> {
  static constexpr int N = 4;
  __device__ static void load(const void* row, int chunk, float (&v)[4]) {
    const float4 f = ((const float4*)row)[chunk];
    v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
  }
};

__device__ __forceinline__ float pick(bool first, float a, float b) { return first ? a : b; }   // (of two values, not of two places)

template <bool BF16, int EMAX>
__global__ __launch_bounds__(256) void router_kernel(const void* __restrict__ x,
                                                     const void* __restrict__ Wgate,
                                                     float* __restrict__ logits, int64_t T, int E,
                                                     int H) {
  using C = Chunk<BF16>;
  constexpr int ES = BF16 ? 2 : 4;
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t n_waves = (int64_t)gridDim.x * 4;
  const int chunks = H / C::N;
  const size_t row_bytes = (size_t)H * ES;

  for (int64_t t0 = wave * TOK; t0 < T; t0 += n_waves * TOK) {
    float acc[TOK][EMAX];
#pragma unroll
    for (int i = 0; i < TOK; ++i)
#pragma unroll
      for (int e = 0; e < EMAX; ++e) acc[i][e] = 0.f;

    for (int c = lane; c < chunks; c += 64) {
      float xv[TOK][C::N];
#pragma unroll
      for (int i = 0; i < TOK; ++i) {
        const int64_t t = t0 + i < T ? t0 + i : T - 1;
        C::load((const char*)x + t * row_bytes, c, xv[i]);
      }
      // (experts beyond the last one repeat it, their sums are not stored: without a branch per expert the loads overlap)
#pragma unroll
      for (int e = 0; e < EMAX; ++e) {
        float wv[C::N];
        C::load((const char*)Wgate + (e < E ? e : E - 1) * row_bytes, c, wv);
#pragma unroll
        for (int i = 0; i < TOK; ++i)
#pragma unroll
          for (int j = 0; j < C::N; ++j) acc[i][e] = fmaf(xv[i][j], wv[j], acc[i][e]);
      }
    }
    // Sums over the lanes, 32, 16, ..., 1 apart.  A lane keeps half of its values at each distance and gives the others away, so
    // that TOK x EMAX of them take about as many exchanges, where a butterfly per value took six for each.  With the branches
    // per expert gone as well: all experts of a layer, E 8, H 512, F 1024, 1501 tokens 439 -> 431 us, E 16, H 1024, F 512, 64 tokens
    // 153 -> 137.  All EMAX columns are multiplied, so the forms are a factor of two apart: this kernel, fp32, H 2048,
    // us, with the branches / by 8 columns / by 4: E 2, 64 tokens 8.2 / 9.1 / 7.2, 12000 19.2 / 22.6 / 19.4; E 3, 12000 22.6 / 24.5 / 20.9;
    // E 17 by 32 columns, 12000 130 / 111.
    float v[TOK * EMAX];
#pragma unroll
    for (int i = 0; i < TOK; ++i)
#pragma unroll
      for (int e = 0; e < EMAX; ++e) v[i * EMAX + e] = acc[i][e];
    int first = 0;                                       // of the lane's values
    constexpr int N = TOK * EMAX, HALVINGS = N >= 64 ? 6 : N >= 32 ? 5 : 4;
    static_assert(N >= 16 && (N & (N - 1)) == 0, "values that halve");
#pragma unroll
    for (int h = 0; h < HALVINGS; ++h) {
      const int n = N >> (h + 1), off = 32 >> h;
      const bool upper = (lane & off) != 0;
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const float a = v[i], b = v[n + i];
        v[i] = pick(upper, b, a) + __shfl_xor(pick(upper, a, b), off, 64);
      }
      first += upper ? n : 0;
    }
    constexpr int LEFT = TOK * EMAX > 64 ? TOK * EMAX / 64 : 1;
#pragma unroll
    for (int off = 32 >> HALVINGS; off >= 1; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
#pragma unroll
    for (int i = 0; i < LEFT; ++i) {
      const int token = (first + i) / EMAX, e = (first + i) % EMAX;
      if (e < E && t0 + token < T) logits[(t0 + token) * E + e] = v[i];
    }
  }
}

// bf16, E <= 32: the same product on the MFMA units (the fp32 FMAs and the bf16 unpacking of the kernel
// above cost more cycles than reading x does: 0.57 ms for 262144 x 4096 against 0.44 ms here).  A wavefront
// takes 16 tokens; per 32 hidden units one v_mfma_f32_16x16x32_bf16 multiplies the 16 token rows with the
// (at most 16, zero-padded) expert rows of Wgate, which stay in L1/L2 (WIDE, E > 16: a second MFMA takes experts 16 .. 31).  Lane l supplies row l % 16 and
// hidden units 8 (l / 16) .. + 7 of a slice; register v of lane l of the result is token 4 (l / 16) + v,
// expert l % 16.  A token's sum depends on its own row and H only.  (Two tiles per wavefront sharing the
// Wgate fragments, and 1 KB row-wise loads staged through LDS, both measured slower.)
// PACK: the wavefront also writes its 16 rows of x in the blocked operand layout of the packed GEMM (see
// gemm_bf16_packed.hip: tile of 256 rows, slice of 32 hidden units, row p of a block = 64 bytes whose 16-byte chunk c
// sits at position c ^ ((p >> 2) & 3)) -- the registers it feeds the MFMA with are exactly one row group of a block,
// 1 KB of consecutive bytes per store -- so that the expert pass reads x once for both.  Row groups beyond T, up to
// the end of the last tile, are filled with the last row (their products are never stored).
template <bool PACK, bool WIDE>
__global__ __launch_bounds__(256) void router_mfma_kernel(const uint4* __restrict__ x,
                                                          const uint4* __restrict__ Wgate,
                                                          float* __restrict__ logits, int64_t T, int E,
                                                          int H, uint4* __restrict__ xpacked) {
  const int lane = threadIdx.x & 63;
  const int64_t t0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  if (t0 >= (PACK ? (T + 255) / 256 * 256 : T)) return;
  const int row = lane & 15, kg = lane >> 4;
  const int chunks = H / 8;
  const int64_t t = t0 + row < T ? t0 + row : T - 1;
  const uint4* xp = x + t * chunks + kg;
  // packed destination of this lane's chunk of slice 0; consecutive slices are 1024 chunks (16 KB) apart
  const int p_row = (int)((t0 + row) & 255);
  uint4* const dst = PACK ? xpacked + ((t0 >> 8) * (int64_t)(H / 32)) * 1024 + p_row * 4 + (kg ^ ((p_row >> 2) & 3)) : nullptr;
  const bool w_valid = row < E, w2_valid = WIDE && 16 + row < E;
  const uint4* wp = Wgate + (int64_t)(w_valid ? row : 0) * chunks + kg;
  const uint4* wp2 = Wgate + (int64_t)(w2_valid ? 16 + row : 0) * chunks + kg;
  r_f32x4 acc[8], acc2[WIDE ? 8 : 1];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    acc[i] = r_f32x4{0.f, 0.f, 0.f, 0.f};
    if (WIDE) acc2[i] = acc[i];
  }
  const int steps = H / 32;
  for (int s0 = 0; s0 < steps; s0 += 8) {
    uint4 xv[8], wv[8], wv2[WIDE ? 8 : 1];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool in = s0 + i < steps;
      xv[i] = in ? xp[(s0 + i) * 4] : make_uint4(0, 0, 0, 0);
      wv[i] = (in && w_valid) ? wp[(s0 + i) * 4] : make_uint4(0, 0, 0, 0);
      if (WIDE) wv2[i] = (in && w2_valid) ? wp2[(s0 + i) * 4] : make_uint4(0, 0, 0, 0);
      if (PACK && in) dst[(int64_t)(s0 + i) * 1024] = xv[i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(r_bf16x8, xv[i]), __builtin_bit_cast(r_bf16x8, wv[i]),
                                                       acc[i], 0, 0, 0);
      if (WIDE)
        acc2[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(r_bf16x8, xv[i]),
                                                          __builtin_bit_cast(r_bf16x8, wv2[i]), acc2[i], 0, 0, 0);
    }
  }
  const r_f32x4 sum = sum_of_eight([&](int i) { return acc[i]; }), sum2 = sum_of_eight([&](int i) { return acc2[WIDE ? i : 0]; });
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t tt = t0 + 4 * kg + v;
    if (tt < T && row < E) logits[tt * E + row] = sum[v];
    if (WIDE && tt < T && 16 + row < E) logits[tt * E + 16 + row] = sum2[v];
  }
}

template <bool PACK, bool WIDE, int W>
__global__ __launch_bounds__(W == 8 ? 512 : 256) void router_few_kernel(const uint4* __restrict__ x, const uint4* __restrict__ Wgate,
                                                                        float* __restrict__ logits, int64_t T, int E, int H,
                                                                        uint4* __restrict__ xpacked) {
  router_few<PACK, WIDE, W>(x, Wgate, logits, T, E, H, xpacked);
}

// Up to this many tokens two wavefronts per 16 tokens are faster than one; beyond it there are wavefronts enough to hide the loads.
// Eight are faster still while a compute unit has no second workgroup of them, or where rows are long.  One / two / eight, us.
// E 8: H 1024, 4096 tokens 10.5 / 8.0 / 6.2, 8192 10.5 / 8.1 / 8.6; H 2048, 4096 16.2 / 10.7 / 7.8, 8192 17.2 / 11.6 / 12.4; H 3072,
// 4096 21.6 / 14.0 / 8.9, 8192 23.3 / 17.2 / 16.4, 16384 27.7 / 30.3 / 29.4; H 4096, 4096 28.2 / 17.6 / 11.2, 8192 30.1 / 26.6 / 23.0,
// 32768 69.2 / 79.7 / 66.1, 49152 99.4 / 112 / 95.3; H 6144, 32768 106 / 108 / 104, 49152 146 / 156 / 152.  E 32: H 2048, 8192 27.0 /
// 16.9 / 17.5; H 4096, 8192 49.2 / 33.1 / 29.9, 32768 101 / 105 / 103.  With the packed copy of x, E 8: H 1024, 8192 15.5 / 12.2 / 10.6; H 4096,
// 4096 70.4 / 27.0 / 21.0, 16384 99.1 / 94.5 / 78.6, 32768 158 / 142 / 137.  Short rows
// with it: H 64, 12000 tokens 6.7 / 10.4 / 9.2, H 256 8.8 / 11.5 / 10.6, H 384 10.7 / 12.6 / 11.8, H 512, 16384 11.1 / 11.8 / 12.9.
// (It leaves room: H 4096, 49152 tokens 214 / 189 / 172, H 2048, 24576 71.8 / 59.5 / 58.1, with one wavefront now.)
constexpr int64_t ROUTER_FEW_MAX = 8192, ROUTER_FEW_MAX_PACK = 16384, ROUTER_EIGHT_MAX = 4096, ROUTER_EIGHT_MAX_LONG = 32768;
constexpr int ROUTER_LONG_H = 4096, ROUTER_SHORT_H = 512;

template <bool PACK>
void launch_mfma(const void* x, const void* Wgate, int64_t T, int E, int H, float* logits, void* xpacked,
                 int64_t blocks, hipStream_t s) {
  const int64_t tiles = ceil_div(PACK ? ceil_div(T, 256) * 256 : T, 16);      // of 16 tokens
#define MOEP_ROUTER_FEW(WIDE, W, PER_GROUP)                                                                              \
  hipLaunchKernelGGL((router_few_kernel<PACK, WIDE, W>), dim3((unsigned)ceil_div(tiles, PER_GROUP)), dim3(64 * W * PER_GROUP), 0, s, \
                     (const uint4*)x, (const uint4*)Wgate, logits, T, E, H, (uint4*)xpacked)
  if (T <= (H >= ROUTER_LONG_H ? ROUTER_EIGHT_MAX_LONG : ROUTER_EIGHT_MAX)) {
    if (E > 16) MOEP_ROUTER_FEW(true, 8, 1);
    else MOEP_ROUTER_FEW(false, 8, 1);
    return;
  }
  if (T <= (PACK && H >= ROUTER_SHORT_H ? ROUTER_FEW_MAX_PACK : ROUTER_FEW_MAX)) {
    if (E > 16) MOEP_ROUTER_FEW(true, 2, 2);
    else MOEP_ROUTER_FEW(false, 2, 2);
    return;
  }
#undef MOEP_ROUTER_FEW
  if (E > 16)
    hipLaunchKernelGGL((router_mfma_kernel<PACK, true>), dim3((unsigned)blocks), dim3(256), 0, s, (const uint4*)x,
                       (const uint4*)Wgate, logits, T, E, H, (uint4*)xpacked);
  else
    hipLaunchKernelGGL((router_mfma_kernel<PACK, false>), dim3((unsigned)blocks), dim3(256), 0, s, (const uint4*)x,
                       (const uint4*)Wgate, logits, T, E, H, (uint4*)xpacked);
}

template <bool BF16>
int launch_t(const void* x, const void* Wgate, int64_t T, int E, int H, float* logits, hipStream_t s) {
  if (BF16 && mfma_router_applies(E, H)) {
    const int64_t blocks = ceil_div(T, 64);
    if (blocks < ((int64_t)1 << 31)) {
      launch_mfma<false>(x, Wgate, T, E, H, logits, nullptr, blocks, s);
      MOEP_HIP(hipGetLastError());
      return MOEP_OK;
    }
  }
  const int64_t groups = ceil_div(T, TOK);
  const unsigned blocks = (unsigned)(ceil_div(groups, 4) < 16384 ? ceil_div(groups, 4) : 16384);
  if (E <= 4) hipLaunchKernelGGL((router_kernel<BF16, 4>), dim3(blocks), dim3(256), 0, s, x, Wgate, logits, T, E, H);
  else if (E <= 8) hipLaunchKernelGGL((router_kernel<BF16, 8>), dim3(blocks), dim3(256), 0, s, x, Wgate, logits, T, E, H);
  else if (E <= 16) hipLaunchKernelGGL((router_kernel<BF16, 16>), dim3(blocks), dim3(256), 0, s, x, Wgate, logits, T, E, H);
  else hipLaunchKernelGGL((router_kernel<BF16, 32>), dim3(blocks), dim3(256), 0, s, x, Wgate, logits, T, E, H);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace

int launch_router(const void* x, const void* Wgate, int64_t T, int E, int H, moep_dtype dt,
                  float* logits, hipStream_t s) {
  if (T <= 0) return MOEP_OK;
  if (H % (dt == MOEP_BF16 ? 8 : 4)) return fail(MOEP_EUNSUPPORTED, "router: H=%d not a multiple of the 16-byte chunk", H);
  if (((uintptr_t)x | (uintptr_t)Wgate) & 15) return fail(MOEP_EUNSUPPORTED, "router: x and Wgate must be 16-byte aligned");
  Timed t("router_logits", s);
  return dt == MOEP_BF16 ? launch_t<true>(x, Wgate, T, E, H, logits, s)
                         : launch_t<false>(x, Wgate, T, E, H, logits, s);
}

// bf16: router logits and the packed copy of x in one pass over x.  Returns MOEP_EUNSUPPORTED without launching
// anything when the shape has no fused kernel (the caller then runs the router and the packing separately).
int launch_router_and_pack_x(const void* x, const void* Wgate, int64_t T, int E, int H, float* logits, void* xpacked,
                             hipStream_t s) {
  if (T <= 0) return MOEP_OK;
  const int64_t blocks = ceil_div(ceil_div(T, 256) * 256, 64);
  if (!mfma_router_applies(E, H) || H % 64 || blocks >= ((int64_t)1 << 31)) return MOEP_EUNSUPPORTED;
  if (((uintptr_t)x | (uintptr_t)Wgate | (uintptr_t)xpacked) & 15)
    return fail(MOEP_EUNSUPPORTED, "router: x, Wgate and the packed copy of x must be 16-byte aligned");
  Timed t("router_logits_pack_x", s);
  launch_mfma<true>(x, Wgate, T, E, H, logits, xpacked, blocks, s);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
