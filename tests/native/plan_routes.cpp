// Prints which kernels a compression pass of given sizes takes: one line of numbers per input line "L Hq Hkv d T W B dtype
// flags n_seqs".  Linked with meda_api.hip alone; nothing is launched.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../../paper_2502_17599_amd/csrc/plan.hpp"

namespace meda {
#define MEDA_STUB(name) \
  hipError_t name(const Plan&, const Buffers&, hipStream_t) { abort(); }
MEDA_STUB(launch_score_stats)
MEDA_STUB(launch_stats_combine)
MEDA_STUB(launch_score_accum)
MEDA_STUB(launch_allocate)
MEDA_STUB(launch_select)
MEDA_STUB(launch_similarity)
MEDA_STUB(launch_segment_sort)
MEDA_STUB(launch_merge_write)
}  // namespace meda

int main() {
  meda_params p;
  memset(&p, 0, sizeof p);
  p.recent_num = 3;
  p.recent_den = 4;
  long long budget;
  while (scanf("%d %d %d %d %d %d %lld %d %d %d", &p.n_layers, &p.n_q_heads, &p.n_kv_heads, &p.head_dim, &p.seq_len, &p.window,
               &budget, &p.dtype, &p.flags, &p.n_seqs) == 10) {
    p.total_budget = budget;
    meda::Plan pl;
    const meda_status st = meda::make_plan(&p, &pl);
    if (st != MEDA_OK) printf("status %d\n", (int)st);
    else printf("%d %d %d %d %d %d %d %d\n", pl.direct, pl.blocks, pl.RB, pl.RBa, pl.NQ, pl.NCG * pl.CS, pl.n_blocks_a, pl.sim);
  }
  return 0;
}
