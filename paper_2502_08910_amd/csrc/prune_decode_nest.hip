// Several decode stages scored together over bf16 and E4M3 keys (kernel in prune_decode_nest.h).
#include "prune_decode_nest.h"

namespace ihip {

// K through strides or pages; rope: relative style, or nullptr
void launch_prune_decode_nest(const PruneArgs &a, const NestArgs &nest, int P, bool fp8, const RopeView *rope, int64_t max_seq_len, hipStream_t st)
{
    const RopeView none{nullptr, nullptr, 0};
    if (rope && fp8) launch_nest<true, true>(a, nest, *rope, P, max_seq_len, st);
    else if (rope) launch_nest<true, false>(a, nest, *rope, P, max_seq_len, st);
    else if (fp8) launch_nest<false, true>(a, nest, none, P, max_seq_len, st);
    else launch_nest<false, false>(a, nest, none, P, max_seq_len, st);
}

}  // namespace ihip
