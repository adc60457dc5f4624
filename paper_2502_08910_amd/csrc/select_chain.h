// All stages' selections in one launch (select_chain.hip)
#pragma once

#include "block_select.h"

namespace ihip {

constexpr int kChainMaxStages = 4;
constexpr int kChainMaxScores = 16384;    // of a problem, all stages
constexpr int kChainMaxSlots = 2048;      // candidates of one selection: four to each of 512 threads; larger plans run stage by stage
constexpr int kChainMaxKeep = 2048;
constexpr int kChainMaxParents = 2048;

struct ChainPlan {
    int n_stages;
    int pool;                             // 1, or Hkv: one selection for all KV heads of a sequence (scores max-pooled)
    const float *scores;                  // [P][stride]: per stage the scores of all chunks of the middle range, or of the parents
    int stride;
    int at[kChainMaxStages];              // where a stage's scores begin, multiples of 64
    // per stage: where the list goes, scores, children per parent, chunk size, most kept
    int32_t *out[kChainMaxStages];
    int slots[kChainMaxStages], ratio_log2[kChainMaxStages], chunk[kChainMaxStages], keep[kChainMaxStages];
};

// Stages that select among the keys of chunks kept before: those chunks, of 1 << log2 keys each; starts null: stages of the middle range
struct ChainParents {
    const int32_t *starts;                // [P][n]
    int n, log2;
};

int32_t launch_select_chain(const ihip_shape &s, const ChainPlan &plan, const ChainParents &parents, hipStream_t st);

}  // namespace ihip
