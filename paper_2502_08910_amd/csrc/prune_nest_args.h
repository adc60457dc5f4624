// All stages of a decode plan scored together (prune_decode_nest.h): where the scores go
#pragma once

namespace ihip {

constexpr int kNestLevels = 7;            // chunks of 4, 8, 16, 32, 64, 128 and 256 keys
struct NestArgs {
    float *out[kNestLevels];              // problem 0's scores of the stage with chunks of 4 << level, or null
    int slots[kNestLevels];
    int stride;                           // a problem's scores of all the stages, one after the other
    int top;                              // level of the first stage
};

}  // namespace ihip
