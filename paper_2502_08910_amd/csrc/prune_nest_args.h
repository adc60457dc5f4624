// Several decode stages scored together (prune_decode_nest.h): where their scores go
#pragma once

namespace ihip {

constexpr int kNestLevels = 5;            // chunks of 4, 8, 16, 32 and 64 keys
struct NestArgs {
    float *out[kNestLevels];              // problem 0's scores of the stage with chunks of 4 << level, or null
    int slots[kNestLevels];
    int stride;                           // a problem's scores of all the stages, one after the other
    int top;                              // level of the first of the stages; PruneArgs describes that one
};

}  // namespace ihip
