// Triangle, 4-cycle and 4-clique counts of the pairwise graph without bit
// rows (wedge.hip).
#pragma once

#include "hm_internal.h"

namespace hm {

// counters many workgroups add to are kept in this many copies
constexpr uint32_t kAccCopies = 16;

int wedge_counts(hm_graph* H, int k, uint32_t* tri_e, unsigned long long* n_cycles, unsigned long long* n_cliques,
                 hipStream_t st);
int wedge_edge_stats(hm_graph* H, unsigned long long* es, hipStream_t st);

}  // namespace hm
