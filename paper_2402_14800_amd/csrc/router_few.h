// The router on the matrix units for few tokens, as a device function: a kernel of its own (router.hip), and the first half of the
// kernel that routes a handful of tokens (skip.hip).
#pragma once

#include "common.h"

namespace moep {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 r_bf16x8;
typedef __attribute__((ext_vector_type(4))) float r_f32x4;
// The sums of the slices 0, 8, ..., of 1, 9, ..., up to 7, 15, ..., added four, two and one apart: the order of every kernel here.
template <class F>
__device__ __forceinline__ r_f32x4 sum_of_eight(F part) {
  return ((part(0) + part(4)) + (part(2) + part(6))) + ((part(1) + part(5)) + (part(3) + part(7)));
}

// router_mfma_kernel (router.hip) for few tokens, where a wavefront's serial walk over H is all there is (27 us for 777 tokens of H =
// 4096, 11 for one): W = 2 or 8 wavefronts share 16 tokens, wavefront w takes the slices w, w + W, ..., each with 32 or 16 of them in
// flight, and the eight sums are added at the end -- the sums of that kernel, bit for bit.
// The workgroup has 64 W wavefront lanes per 16 tokens: 512 threads and 16 tokens (W = 8) or 256 and 32.
template <bool PACK, bool WIDE, int W>
__device__ __forceinline__ void router_few(const uint4* __restrict__ x, const uint4* __restrict__ Wgate, float* __restrict__ logits,
                                           int64_t T, int E, int H, uint4* __restrict__ xpacked) {
  constexpr int B = W == 8 || WIDE ? 8 : 16;              // slices per batch, two batches in registers
  constexpr int SUMS = 8 / W, TILES = W == 8 ? 1 : 2, PARTS = WIDE ? 2 : 1;
  __shared__ r_f32x4 part[TILES][8][PARTS][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = wave / W, w = wave % W;
  const int64_t t0 = ((int64_t)blockIdx.x * TILES + tile) * 16;
  const bool active = t0 < (PACK ? (T + 255) / 256 * 256 : T);
  const int row = lane & 15, kg = lane >> 4;
  const int chunks = H / 8;
  const int64_t t = t0 + row < T ? t0 + row : T - 1;
  const uint4* xp = x + t * chunks + kg + w * 4;
  const int p_row = (int)((t0 + row) & 255);
  uint4* const dst = PACK ? xpacked + ((t0 >> 8) * (int64_t)(H / 32) + w) * 1024 + p_row * 4 + (kg ^ ((p_row >> 2) & 3)) : nullptr;
  const bool w_valid = row < E, w2_valid = WIDE && 16 + row < E;
  const uint4* wp = Wgate + (int64_t)(w_valid ? row : 0) * chunks + kg + w * 4;
  const uint4* wp2 = Wgate + (int64_t)(w2_valid ? 16 + row : 0) * chunks + kg + w * 4;
  const int n = (H / 32 - w + W - 1) / W;                 // slices w, w + W, ...: the i-th belongs to sum w + W (i % SUMS)
  r_f32x4 acc[SUMS], acc2[SUMS];
#pragma unroll
  for (int i = 0; i < SUMS; ++i) acc[i] = acc2[i] = r_f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 xv[2][B], wv[2][B], wv2[2][WIDE ? B : 1];
  auto fetch = [&](int set, int i0) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const bool in = i0 + i < n;
      xv[set][i] = in ? xp[(int64_t)(i0 + i) * (4 * W)] : make_uint4(0, 0, 0, 0);
      wv[set][i] = (in && w_valid) ? wp[(int64_t)(i0 + i) * (4 * W)] : make_uint4(0, 0, 0, 0);
      if (WIDE) wv2[set][i] = (in && w2_valid) ? wp2[(int64_t)(i0 + i) * (4 * W)] : make_uint4(0, 0, 0, 0);
    }
  };
  auto use = [&](int set, int i0) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      if (PACK && i0 + i < n) dst[(int64_t)(i0 + i) * (1024 * W)] = xv[set][i];
      acc[i % SUMS] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(r_bf16x8, xv[set][i]),
                                                              __builtin_bit_cast(r_bf16x8, wv[set][i]), acc[i % SUMS], 0, 0, 0);
      if (WIDE)
        acc2[i % SUMS] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(r_bf16x8, xv[set][i]),
                                                                 __builtin_bit_cast(r_bf16x8, wv2[set][i]), acc2[i % SUMS], 0, 0, 0);
    }
  };
  if (active) {
    fetch(0, 0);
    for (int i0 = 0; i0 < n; i0 += 2 * B) {
      fetch(1, i0 + B);
      use(0, i0);
      fetch(0, i0 + 2 * B);
      use(1, i0 + B);
    }
  }
#pragma unroll
  for (int i = 0; i < SUMS; ++i) {
    part[tile][w + W * i][0][lane] = acc[i];
    if (WIDE) part[tile][w + W * i][PARTS - 1][lane] = acc2[i];
  }
  __syncthreads();
  if (w >= PARTS || !active) return;                      // a wavefront per 16 experts adds them
  const r_f32x4 sum = sum_of_eight([&](int i) { return part[tile][i][w][lane]; });
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t tt = t0 + 4 * kg + v;
    if (tt < T && 16 * w + row < E) logits[tt * E + 16 * w + row] = sum[v];
  }
}

}  // namespace

inline bool mfma_router_applies(int E, int H) { return E <= 32 && H % 32 == 0; }

}  // namespace moep
