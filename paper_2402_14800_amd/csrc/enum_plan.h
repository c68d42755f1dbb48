// The plan of a subset enumeration.  Host arithmetic only, without HIP, so that a program built on the CPU can check it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace moep {

struct EnumPlan {
  int64_t T; int E, H, k, r;
  int kk;            // min(k, r): experts per token in the pruned layer
  int n_act;         // min(E, kk + E - r): rank positions that can be selected
  int64_t n_sub;     // C(E, r)
  int rec_floats;    // floats per token record
  int tok_tile;      // tokens per scoring block
  int64_t n_tok_tiles;
  bool use_lut;      // many subsets, few selections per token: score through per-token selection tables
  int n_combo;       // C(n_act, kk): selections per token
  int fused_threads; // up to 16 experts: tables and look-ups in one kernel, its workgroup (0: not taken),
  int fused_spl;     //   subsets per lane,
  int fused_tg;      //   tokens per barrier
  size_t fused_lds;  //   and dynamic LDS
  // workspace carving (byte offsets)
  size_t off_gram, off_rec, off_masks, off_partial, off_partial_cnt, off_qtab, off_sel, off_selbits, off_nib, total;
};
int plan_enumerate(int64_t T, int E, int H, int k, int r, EnumPlan* p);

}  // namespace moep
