// Numbering of the sets of nodes and of their rows, for the searches by subsets of up to PPO_MAX_K nodes.
#pragma once

#include "ppo_common.h"

namespace ppo {

// Sets of up to 12 nodes in increasing order of their size, then of their value (so that the first C(k, c) of size c
// are those of the first k nodes), and the number of the first row of every set: rows are numbered set by set in
// numeric order, member by member (see cluster_first_row in ppo_cluster.hip for the sum).
struct SetTables {
    uint32_t order[1 << PPO_MAX_K];       // set | first row << 16
    int first[PPO_MAX_K + 2];             // first entry of every size
    uint32_t choose[PPO_MAX_K + 1][PPO_MAX_K + 1];
    constexpr SetTables() : order{}, first{}, choose{} {
        for (int i = 0; i <= PPO_MAX_K; ++i) {
            choose[i][0] = 1;
            for (int j = 1; j <= i; ++j) choose[i][j] = choose[i - 1][j - 1] + (j <= i - 1 ? choose[i - 1][j] : 0u);
        }
        int at[PPO_MAX_K + 2] = {};
        for (int c = 0; c <= PPO_MAX_K; ++c) first[c + 1] = first[c] + (int)choose[PPO_MAX_K][c];
        for (int c = 0; c <= PPO_MAX_K + 1; ++c) at[c] = first[c];
        uint32_t rows = 0;
        for (uint32_t s = 0; s < (1u << PPO_MAX_K); ++s) {
            int c = 0;
            for (uint32_t b = s; b; b &= b - 1u) ++c;
            order[at[c]++] = s | (rows << 16);
            rows += (uint32_t)c;
        }
    }
};
constexpr SetTables kSetsHost = SetTables();
static __constant__ SetTables kSets = SetTables();   // one for each file that includes this
static_assert((PPO_MAX_K << (PPO_MAX_K - 1)) < 65536, "a row's number fits 16 bits");

// The same by the value of a set: its first row | its place among the sets of its size << 16; and where the sets of every
// size start, in increasing order of size, among those of k nodes.
struct SetValues {
    uint32_t row_and_place[1 << PPO_MAX_K];
    uint32_t level[PPO_MAX_K + 1][PPO_MAX_K + 2];
    constexpr SetValues() : row_and_place{}, level{} {
        const SetTables by_size;
        for (int c = 0; c <= PPO_MAX_K; ++c)
            for (int i = by_size.first[c]; i < by_size.first[c + 1]; ++i)
                row_and_place[by_size.order[i] & 0xFFFFu] = (by_size.order[i] >> 16) | ((uint32_t)(i - by_size.first[c]) << 16);
        for (int k = 0; k <= PPO_MAX_K; ++k)
            for (int c = 0; c <= k; ++c) level[k][c + 1] = level[k][c] + by_size.choose[k][c];
    }
};

__device__ __forceinline__ uint32_t row_of(uint32_t set_first_row, uint32_t mp, uint32_t j) {
    // first row of R' + j from the first row of R' (j not in R'), then j's place among the members
    const uint32_t below = mp & ((1u << j) - 1u);
    const uint32_t above = (uint32_t)__popc((mp >> j) >> 1);
    return set_first_row + (above << j) + ((j << j) >> 1) + below + (uint32_t)__popc(below);
}

}  // namespace ppo
