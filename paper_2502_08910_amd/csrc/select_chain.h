// All stages' selections in one launch (select_chain.hip)
#pragma once

#include "block_select.h"

namespace ihip {

constexpr int kChainMaxStages = 4;
constexpr int kChainMaxScores = 16384;    // of a problem, all stages
constexpr int kChainMaxSlots = 2048;      // candidates of one selection: four to each of 512 threads; larger plans run stage by stage
constexpr int kChainMaxKeep = 2048;

struct ChainPlan {
    int n_stages;
    int pool;                             // 1, or Hkv: one selection for all KV heads of a sequence (scores max-pooled)
    const float *scores;                  // [P][stride]: per stage the scores of all chunks of the middle range
    int stride;
    int at[kChainMaxStages];              // where a stage's scores begin, multiples of 64
    // per stage: where the list goes, scores, children per parent, chunk size, most kept
    int32_t *out[kChainMaxStages];
    int slots[kChainMaxStages], ratio_log2[kChainMaxStages], chunk[kChainMaxStages], keep[kChainMaxStages];
};

int32_t launch_select_chain(const ihip_shape &s, const ChainPlan &plan, hipStream_t st);

}  // namespace ihip
