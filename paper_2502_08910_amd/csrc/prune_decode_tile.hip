// Decode pruning stages on the matrix cores over bf16 and E4M3 keys (kernels in prune_decode_tile.h).
#include "prune_decode_tile.h"

namespace ihip {

// K through strides or pages, four or eight heads (E4M3 rows: any number; the caller checks); rope: relative style, or nullptr
void launch_prune_decode_tile(const PruneArgs &a, int P, bool fp8, const RopeView *rope, int64_t max_seq_len, hipStream_t st)
{
    const RopeView none{nullptr, nullptr, 0};
    if (rope && fp8) launch_decode_tile<true, true>(a, *rope, P, max_seq_len, st);
    else if (rope) launch_decode_tile<true, false>(a, *rope, P, max_seq_len, st);
    else if (fp8) launch_decode_tile<false, true>(a, none, P, max_seq_len, st);
    else launch_decode_tile<false, false>(a, none, P, max_seq_len, st);
}

// any group size, K behind the host tier
void launch_prune_decode_tile_cached(const PruneArgs &a, int P, bool fp8, const RopeView *rope, hipStream_t st)
{
    const RopeView none{nullptr, nullptr, 0};
    if (rope && fp8) launch_decode_tile_cached<true, true>(a, *rope, P, st);
    else if (rope) launch_decode_tile_cached<true, false>(a, *rope, P, st);
    else if (fp8) launch_decode_tile_cached<false, true>(a, none, P, st);
    else launch_decode_tile_cached<false, false>(a, none, P, st);
}

}  // namespace ihip
