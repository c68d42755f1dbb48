// Calibration of the skipping threshold (Sec. 3.3; appendix on experiment details): beta is the
// median over the calibration tokens of w_e1 / w_e0 = exp(l_e1 - l_e0), e0 and e1 being the token's
// top-2 experts (among the kept ones).  exp is monotone, so the two middle order statistics of
// delta = l_e1 - l_e0 (fp32, the same subtraction the routing kernel thresholds) are selected
// exactly by a most-significant-digit radix select on the order-preserving integer image of the
// floats, and beta = (exp(delta_lo) + exp(delta_hi)) / 2 is formed in fp64 at the very end.
//
//   select_one  few tokens: everything in one workgroup, the keys in LDS.
//   keys        more tokens: one thread per token: top-2 (ties -> lower index), delta, key; block 0 also clears
//               the histograms (a kernel rather than a memset so that the call can be graph-captured)
//   hist        3 passes of 11, 11 and 10 bits: every workgroup first finds, from the finished histogram of the pass
//               before, the digit that holds each wanted rank (the same integers in all of them; block 0 notes them
//               for the pass after), then counts the keys that match the digits chosen so far (integer atomics only:
//               order-independent)
//   finish      the last digit, the two keys turned back into floats, beta
//
// Nothing here is bound by bytes (a million tokens are 32 MB of logits): it is launches and the serial walk over a
// histogram.  4 passes of 8 bits with a one-thread walk between them took 9 launches and 45 to 90 us at any size.
// Measured (E 8), before and after: 2048 tokens 65 -> 12 us, 16384 56 -> 19 us, 262144 70 -> 30 us.
#include <cmath>

#include "common.h"

namespace moep {
namespace {

constexpr int CB = 256;            // threads of the multi-workgroup kernels
// select_one: at most 8192 tokens (8 per thread, their keys 32 KB of LDS), and as many logits as one compute unit reads as
// fast as the other form launches its kernels.  That depends on how it reads them: rows in 16-byte pieces; word by word; word
// by word with rows a multiple of 32 bytes apart, where a wavefront's words crowd into few sets of the L1.  Just outside the
// line on the left, inside it on the right, one launch / five, us on logits just written:
//   pieces, E <= 16   6000 x 16 19 / 19           4096 x 16 16 / 18,  8192 x 8 15 / 18
//   pieces, E > 16    3276 x 20 21.9 / 18.8, 2048 x 32 20.4 / 19.4    2457 x 20 18.1 / 18.5, 1755 x 28 18 / 19
//   words, E <= 16    7021 x 7 17.3 / 17.1, 5461 x 9 19.3 / 17.8      4444 x 9 17.3 / 17.8,  5714 x 7 14.7 / 17.3
//   words, E > 16     2352 x 17 20.7 / 19.2, 1428 x 28 20.6 / 20.6    1927 x 17 18.5 / 19.5
//   words, 32 bytes   4096 x 8 21.5 / 17.8, 1024 x 32 23.4 / 22.1     2500 x 8 and 625 x 32 faster by more than 1
constexpr int ONE_MAX = 8192;
int64_t one_logits(int E, bool vec) {
  if (vec) return E <= 16 ? 65536 : 49152;
  return E % 8 == 0 ? 24576 : E <= 16 ? 40000 : 32768;
}
constexpr int BITS = 11, BINS = 1 << BITS, PASSES = 3;

struct SelectState {          // per wanted rank q in {0, 1}
  uint32_t prefix[2];         // digits chosen so far, in place
  uint32_t rem[2];            // rank still to find inside the matching keys
};

__device__ __forceinline__ uint32_t float_to_key(float f) {     // ascending floats -> ascending keys
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __builtin_bit_cast(float, u);
}

template <int EMAX>
__device__ __forceinline__ uint32_t token_key(const float* logits, int64_t t, int E, bool vec, uint32_t kept) {
  float v[EMAX];
  load_logits<EMAX>(logits, t, E, vec, v);
  const TopTwo t2 = top_two<EMAX>(v, E, kept);
  return float_to_key(t2.l1 - t2.l0);
}

// Digit p covers bits [shift(p), shift(p) + width): 11, 11 and 10 bits from the top.
__device__ __forceinline__ int digit_shift(int p) { return p == 0 ? 21 : p == 1 ? 10 : 0; }
__device__ __forceinline__ uint32_t digit_bins(int p) { return p == 2 ? 1u << 10 : 1u << BITS; }
__device__ __forceinline__ uint32_t chosen_bits(int p) { return p == 0 ? 0u : p == 1 ? 0xffe00000u : 0xfffffc00u; }

// The bucket of a histogram of BINS counts that holds rank `rem`, and the rank inside it, found by the first BINS / 8
// threads of the workgroup (a multiple of 64 of them); result[0], result[1] for all.  The last bucket takes a rank beyond
// the total.  Ends with a barrier.
__device__ void find_bucket(const uint32_t* h, uint32_t rem, uint32_t* scratch /* BINS / 512 */, uint32_t* result) {
  constexpr int W = BINS / 8 / 64;                // wavefronts
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t c[8], sum = 0, upto = 0;
  if (tid < BINS / 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { c[i] = h[tid * 8 + i]; sum += c[i]; }
    upto = sum;                                   // inclusive sum over the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t v = __shfl_up(upto, off, 64);
      if (lane >= off) upto += v;
    }
    if (lane == 63) scratch[wave] = upto;
  }
  __syncthreads();
  if (tid < BINS / 8) {
    uint32_t before = upto - sum;
    for (int w = 0; w < W; ++w)
      if (w < wave) before += scratch[w];
    const bool last = tid == BINS / 8 - 1;
    if (rem >= before && (rem < before + sum || last)) {
      int d = 0;
      for (; d < 7; ++d) {
        if (before + c[d] > rem) break;
        before += c[d];
      }
      result[0] = (uint32_t)(tid * 8 + d);
      result[1] = rem - before;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ float beta_of(uint32_t key_lo, uint32_t key_hi) {
  const double lo = exp((double)key_to_float(key_lo));
  const double hi = exp((double)key_to_float(key_hi));
  return (float)(0.5 * (lo + hi));
}

template <int EMAX>
__global__ __launch_bounds__(1024) void select_one_kernel(const float* __restrict__ logits, int T, int E, bool vec, uint32_t kept,
                                                          float* __restrict__ beta_out) {
  __shared__ uint32_t keys[ONE_MAX];
  __shared__ uint32_t h[2][BINS];
  __shared__ uint32_t scratch[BINS / 512], found[2][2];
  for (int i = threadIdx.x; i < T; i += 1024) keys[i] = token_key<EMAX>(logits, i, E, vec, kept);
  uint32_t prefix[2] = {0u, 0u}, rem[2] = {(uint32_t)((T - 1) / 2), (uint32_t)(T / 2)};
  for (int p = 0; p < PASSES; ++p) {
    for (int i = threadIdx.x; i < 2 * BINS; i += 1024) (&h[0][0])[i] = 0;
    __syncthreads();
    const bool same = prefix[0] == prefix[1];     // one histogram serves both ranks until they part
    const uint32_t mask = chosen_bits(p);
    const int shift = digit_shift(p);
    for (int i = threadIdx.x; i < T; i += 1024) {
      const uint32_t k = keys[i], d = (k >> shift) & (digit_bins(p) - 1);
      if ((k & mask) == prefix[0]) atomicAdd(&h[0][d], 1u);
      if (!same && (k & mask) == prefix[1]) atomicAdd(&h[1][d], 1u);
    }
    __syncthreads();
    for (int q = 0; q < 2; ++q) find_bucket(h[same ? 0 : q], rem[q], scratch, found[q]);
    for (int q = 0; q < 2; ++q) {
      prefix[q] |= found[q][0] << shift;
      rem[q] = found[q][1];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *beta_out = beta_of(prefix[0], prefix[1]);
}

template <int EMAX>
__global__ __launch_bounds__(CB) void keys_kernel(const float* __restrict__ logits, int64_t T, int E, bool vec,
                                                  uint32_t kept, uint32_t* __restrict__ keys,
                                                  uint32_t* __restrict__ hist) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < PASSES * 2 * BINS; i += CB) hist[i] = 0;
  const int64_t t = (int64_t)blockIdx.x * CB + threadIdx.x;
  if (t < T) keys[t] = token_key<EMAX>(logits, t, E, vec, kept);
}

// The state before pass p, from the one before pass p - 1 and that pass's histogram.
__device__ void state_before(int p, int64_t T, const SelectState* __restrict__ states, const uint32_t* __restrict__ hist,
                             uint32_t* scratch, uint32_t (*found)[2], SelectState* out) {
  if (p == 0) {
    out->prefix[0] = out->prefix[1] = 0;
    out->rem[0] = (uint32_t)((T - 1) / 2);
    out->rem[1] = (uint32_t)(T / 2);
    return;
  }
  for (int q = 0; q < 2; ++q) find_bucket(hist + (size_t)((p - 1) * 2 + q) * BINS, states[p - 1].rem[q], scratch, found[q]);
  for (int q = 0; q < 2; ++q) {
    out->prefix[q] = states[p - 1].prefix[q] | (found[q][0] << digit_shift(p - 1));
    out->rem[q] = found[q][1];
  }
}

__global__ __launch_bounds__(CB) void hist_kernel(const uint32_t* __restrict__ keys, int64_t T, int p,
                                                  SelectState* __restrict__ states, uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[2][BINS];
  __shared__ uint32_t scratch[BINS / 512], found[2][2];
  SelectState st;
  state_before(p, T, states, hist, scratch, found, &st);
  if (blockIdx.x == 0 && threadIdx.x == 0) states[p] = st;
  for (int i = threadIdx.x; i < 2 * BINS; i += CB) (&h[0][0])[i] = 0;
  __syncthreads();
  const bool same = st.prefix[0] == st.prefix[1];
  const uint32_t mask = chosen_bits(p);
  const int shift = digit_shift(p);
  for (int64_t i = (int64_t)blockIdx.x * CB + threadIdx.x; i < T; i += (int64_t)gridDim.x * CB) {
    const uint32_t k = keys[i], d = (k >> shift) & (digit_bins(p) - 1);
    if ((k & mask) == st.prefix[0]) atomicAdd(&h[0][d], 1u);
    if (!same && (k & mask) == st.prefix[1]) atomicAdd(&h[1][d], 1u);
  }
  __syncthreads();
  uint32_t* g = hist + (size_t)p * 2 * BINS;
  for (int i = threadIdx.x; i < BINS; i += CB) {
    const uint32_t lo = h[0][i], hi = same ? lo : h[1][i];
    if (lo) atomicAdd(&g[i], lo);
    if (hi) atomicAdd(&g[BINS + i], hi);
  }
}

__global__ __launch_bounds__(CB) void finish_kernel(int64_t T, const SelectState* __restrict__ states,
                                                    const uint32_t* __restrict__ hist, float* __restrict__ beta_out) {
  __shared__ uint32_t scratch[BINS / 512], found[2][2];
  SelectState st;
  state_before(PASSES, T, states, hist, scratch, found, &st);
  if (threadIdx.x == 0) *beta_out = beta_of(st.prefix[0], st.prefix[1]);
}

static_assert(BINS / 8 <= CB, "find_bucket needs a thread per 8 buckets");

}  // namespace

size_t calibrate_workspace_bytes(int64_t T) {
  return align256((size_t)T * 4) + align256(PASSES * 2 * BINS * 4) + align256(PASSES * sizeof(SelectState));
}

int launch_calibrate_beta(const float* logits, int64_t T, int E, uint32_t kept_mask, float* beta_out,
                          char* ws, hipStream_t s) {
  Timed t("skip_calibrate_beta", s);
  const bool vec = logits_vec(logits, E);
  if (T <= ONE_MAX && T * E <= one_logits(E, vec)) {
#define MOEP_ONE(EMAX) \
  hipLaunchKernelGGL(select_one_kernel<EMAX>, dim3(1), dim3(1024), 0, s, logits, (int)T, E, vec, kept_mask, beta_out)
    if (E <= 8) MOEP_ONE(8);
    else if (E <= 16) MOEP_ONE(16);
    else MOEP_ONE(32);
#undef MOEP_ONE
    MOEP_HIP(hipGetLastError());
    return MOEP_OK;
  }
  uint32_t* keys = (uint32_t*)ws;
  uint32_t* hist = (uint32_t*)(ws + align256((size_t)T * 4));
  SelectState* states = (SelectState*)((char*)hist + align256(PASSES * 2 * BINS * 4));
  const int64_t n_blocks = ceil_div(T, CB);
  const unsigned hist_blocks = (unsigned)(n_blocks < 512 ? n_blocks : 512);
#define MOEP_KEYS(EMAX) \
  hipLaunchKernelGGL(keys_kernel<EMAX>, dim3((unsigned)n_blocks), dim3(CB), 0, s, logits, T, E, vec, kept_mask, keys, hist)
  if (E <= 8) MOEP_KEYS(8);
  else if (E <= 16) MOEP_KEYS(16);
  else MOEP_KEYS(32);
#undef MOEP_KEYS
  for (int p = 0; p < PASSES; ++p)
    hipLaunchKernelGGL(hist_kernel, dim3(hist_blocks), dim3(CB), 0, s, keys, T, p, states, hist);
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(CB), 0, s, T, states, hist, beta_out);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
