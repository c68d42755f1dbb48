// Expert-selection statistics over a calibration set (baselines of Sec. 4.1; appendix on expert
// selection tendency): count[e] = tokens whose top-k contains e, co[i][j] = tokens whose top-k
// contains both i and j, and the activation-frequency baseline's kept set (the r most selected
// experts, lower index first on equal counts).  Integer work throughout, so the result does not
// depend on the order of execution.
//
// A wavefront takes 64 tokens at a time.  Each lane ranks its token's logits; one ballot per expert then gives the set of
// tokens that selected it, and lane p adds popcount(set_i & set_j) to the pairs (i, j) it owns: E ballots and a few
// look-ups per 64 tokens.  (Counting pairs with LDS atomics, k^2 per token into E^2 counters, took 14 to 19 us however few
// the tokens.)  Up to 512 to 2048 tokens (one_max) one workgroup does everything, the kept set included, in one launch instead of three.
// Measured, before and after: E 8, k 2: 512 tokens 21 -> 4 us, 16384 22 -> 8 us, 262144 43 -> 28 us; E 32, 2048 78 -> 25.
#include "common.h"

namespace moep {
namespace {

constexpr int SB_THREADS = 256, ONE_THREADS = 1024;
// Most tokens of the single-workgroup form.  One launch / three, us: E 8, 1500 tokens 7.5 / 11.2, 2048 8.7 / 11.3, 4001 12.1 / 11.3;
// E 16, 1024 13.8 / 15, 2048 20.2 / 15.4; E 32, 512 28 / 29, 1024 37.6 / 29.
constexpr int64_t one_max(int emax) { return emax <= 8 ? 2048 : emax <= 16 ? 1024 : 512; }

__global__ __launch_bounds__(SB_THREADS) void stats_zero_kernel(unsigned long long* count, unsigned long long* co, int E) {
  for (int i = threadIdx.x; i < E * E; i += SB_THREADS) co[i] = 0;
  if ((int)threadIdx.x < E) count[threadIdx.x] = 0;
}

// Kept mask of the r largest counts, by one wavefront: lane e ranks expert e (kept iff fewer than r come before it).
__device__ void most_frequent(const unsigned long long* count, int E, int r, uint32_t* mask_out) {
  const int e = threadIdx.x & 63;
  const unsigned long long mine = e < E ? count[e] : 0;
  int before = 0;
  for (int f = 0; f < E; ++f) {
    const unsigned long long c = __shfl(mine, f, 64);
    before += (c > mine || (c == mine && f < e)) ? 1 : 0;
  }
  const unsigned long long kept = __ballot(e < E && before < r);
  if (e == 0) *mask_out = (uint32_t)kept;
}

// EMAX >= E.  ONE: a single workgroup over all tokens, which writes the outputs (and the kept mask) itself.
template <int EMAX, bool ONE>
__global__ __launch_bounds__(ONE ? ONE_THREADS : SB_THREADS) void stats_kernel(
    const float* __restrict__ logits, int64_t T, int E, bool vec, int k, int r, unsigned long long* __restrict__ count,
    unsigned long long* __restrict__ co, uint32_t* __restrict__ mask_out) {
  constexpr int THREADS = ONE ? ONE_THREADS : SB_THREADS;
  constexpr int PAIRS = EMAX * (EMAX + 1) / 2, OWN = (PAIRS + 63) / 64;
  __shared__ unsigned long long sets[THREADS / 64][EMAX];
  __shared__ unsigned int tab[EMAX][EMAX];
  __shared__ unsigned long long totals[EMAX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t stride = (int64_t)gridDim.x * THREADS;
  float next[EMAX];                          // (the first tokens' logits are on their way during the set-up, the next ones' while these are counted)
  auto fetch = [&](int64_t t0) {
    const int64_t t = t0 + lane < T ? t0 + lane : T - 1;
    load_logits<EMAX>(logits, t, E, vec, next);
  };
  int64_t t0 = (int64_t)blockIdx.x * THREADS + wave * 64;
  if (t0 < T) fetch(t0);
  for (int i = threadIdx.x; i < EMAX * EMAX; i += THREADS) (&tab[0][0])[i] = 0;
  // lane p owns pairs p, p + 64, ... of the upper triangle (i <= j), row by row
  int pi[OWN], pj[OWN];
  unsigned int n[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    int q = o * 64 + lane, i = 0;
    if (q >= PAIRS) q = 0;
    while (q >= EMAX - i) { q -= EMAX - i; ++i; }
    pi[o] = i;
    pj[o] = i + q;
    n[o] = 0;
  }
  __syncthreads();
  for (; t0 < T; t0 += stride) {
    const int64_t t = t0 + lane;
    uint32_t mask = 0;                       // expert e is in the top-k iff fewer than k experts come before it
    float v[EMAX];
#pragma unroll
    for (int e = 0; e < EMAX; ++e) v[e] = next[e];
    if (t0 + stride < T) fetch(t0 + stride);
    if (t < T) {
#pragma unroll
      for (int e = 0; e < EMAX; ++e) {
        int before = 0;
#pragma unroll
        for (int f = 0; f < EMAX; ++f)
          if (f < E) before += (v[f] > v[e]) || (v[f] == v[e] && f < e);
        if (e < E && before < k) mask |= 1u << e;
      }
    }
    unsigned long long mine = 0;             // lane e keeps the set of expert e
#pragma unroll
    for (int e = 0; e < EMAX; ++e) {
      const unsigned long long b = __ballot((mask >> e) & 1u);
      if (lane == e) mine = b;
    }
    // (wavefront-private: its LDS operations complete in order, no barrier is needed)
    if (lane < EMAX) sets[wave][lane] = mine;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int o = 0; o < OWN; ++o) n[o] += (unsigned int)__popcll(sets[wave][pi[o]] & sets[wave][pj[o]]);
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int o = 0; o < OWN; ++o)
    if (o * 64 + lane < PAIRS && n[o]) {
      atomicAdd(&tab[pi[o]][pj[o]], n[o]);
      if (pi[o] != pj[o]) atomicAdd(&tab[pj[o]][pi[o]], n[o]);
    }
  __syncthreads();
  for (int idx = threadIdx.x; idx < E * E; idx += THREADS) {
    const int i = idx / E, j = idx - i * E;
    const unsigned int c = tab[i][j];
    if (ONE) {
      co[idx] = c;
      if (i == j) count[i] = totals[i] = c;
    } else if (c) {
      atomicAdd(&co[idx], (unsigned long long)c);
      if (i == j) atomicAdd(&count[i], (unsigned long long)c);
    }
  }
  if (ONE) {
    __syncthreads();
    if (threadIdx.x < 64 && mask_out) most_frequent(totals, E, r, mask_out);
  }
}

__global__ __launch_bounds__(64) void frequency_mask_kernel(const unsigned long long* __restrict__ count, int E, int r, uint32_t* mask_out) {
  most_frequent(count, E, r, mask_out);
}

template <int EMAX>
void launch(const float* logits, int64_t T, int E, int k, int r, unsigned long long* count, unsigned long long* co,
            uint32_t* mask, hipStream_t s) {
  const bool vec = logits_vec(logits, E);
  if (T <= one_max(EMAX)) {
    hipLaunchKernelGGL((stats_kernel<EMAX, true>), dim3(1), dim3(ONE_THREADS), 0, s, logits, T, E, vec, k, r, count, co, mask);
    return;
  }
  hipLaunchKernelGGL(stats_zero_kernel, dim3(1), dim3(SB_THREADS), 0, s, count, co, E);
  const int64_t want = ceil_div(T, SB_THREADS);
  const unsigned blocks = (unsigned)(want < 1024 ? want : 1024);
  hipLaunchKernelGGL((stats_kernel<EMAX, false>), dim3(blocks), dim3(SB_THREADS), 0, s, logits, T, E, vec, k, r, count, co,
                     (uint32_t*)nullptr);
  if (mask) hipLaunchKernelGGL(frequency_mask_kernel, dim3(1), dim3(64), 0, s, count, E, r, mask);
}

}  // namespace

int launch_selection_stats(const float* logits, int64_t T, int E, int k, int r, int64_t* count, int64_t* co,
                           uint32_t* freq_mask, hipStream_t s) {
  Timed t("selection_stats", s);
  unsigned long long* const c = (unsigned long long*)count;
  unsigned long long* const c2 = (unsigned long long*)co;
  if (E <= 8) launch<8>(logits, T, E, k, r, c, c2, freq_mask, s);
  else if (E <= 16) launch<16>(logits, T, E, k, r, c, c2, freq_mask, s);
  else launch<32>(logits, T, E, k, r, c, c2, freq_mask, s);
  MOEP_HIP(hipGetLastError());
  return MOEP_OK;
}

}  // namespace moep
