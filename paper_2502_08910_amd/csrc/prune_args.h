// Arguments of the pruning-stage kernels (Alg. 2 / Alg. 3), shared by the plain and the
// dynamic-RoPE translation units.
#pragma once

#include "common.h"

namespace ihip {

// Rotary table handed in by the caller: cos and sin of (position x angle of frequency j),
// fp32 [n_pos][d/2].
struct RopeView {
    const float *cos, *sin;
    int n_pos;
};

struct PruneArgs {
    Geometry ge;
    const uint16_t *q; int64_t q_sb, q_sh, q_st;
    const uint16_t *k; int64_t k_sb, k_sh, k_st;
    const int32_t *parent_starts;
    int n_parent, ratio_log2, chunk, max_chunks;
    float *out_scores;
    int32_t *out_rep;
    BankView bank;            // used by the cached instantiations only (K then points to host memory)
    PagedView paged;          // paged instantiations only: K is the page pool, k_sb the page stride
    DecodeGrid grid;          // decode
    float k_scale;            // FP8 instantiations only: the scores are multiplied by it (K strides then
                              // count 2-byte units of the byte rows)
};

// The grid of a decode stage's launch, K behind the host tier or not, in E4M3 or not.  Over bf16 pages a stage that covers more than
// 768K keys of a head keeps the part fastest: dealt out problem by problem, a batch of different lengths ends with a few long
// sequences whose pages are all still to be looked up.  Layers over bf16 pages, 8 KV heads, part / problem fastest (us), runs of
// one length and ragged: 4 sequences of 64K 64.2 / 61.7 and 65.4 / 62.1, 16 of 32K 129.2 / 129.4 and 126.1 / 126.8, 4 of
// 250K 111.5 / 112.0 and 104.8 / 108.3, 12 of 333K 314 / 317 and 279 / 287, 8 of 500K 302 / 301 and 268 / 280.  Contiguous rows of any
// size have no such loss (8 of 500K 303 / 297 and 277 / 276), nor E4M3 in pages (237 / 236 and 221 / 222).
inline DecodeGrid prune_grid(const PruneArgs &a, int P, int per_problem, bool fp8)
{
    const bool long_pages = a.paged.block_table != nullptr && !fp8 &&
                            (int64_t)(P / a.ge.Hkv) * a.max_chunks * a.chunk > (int64_t)3 << 18;
    return decode_grid(a.ge, per_problem, long_pages || a.bank.page_table != nullptr);
}

// Decode on the matrix cores (prune_decode_tile.h): chunks a wave works on, and waves of a workgroup
constexpr int kDecodeTileWaves = 4;
__host__ __device__ constexpr int decode_tile_chunks(int G, int chunk, bool rope, bool fp8)
{
    return chunk == 4 ? (rope && !fp8 ? 8 : 16) : 64 / G;
}

// Chunk-indexed RoPE needs the number of chunks this stage really has for problem p (valid slots are
// a prefix of the slot list: parents are ascending with the empty ones last, and only the last chunk
// before the end of the middle range can be cut short).  Every thread of the workgroup calls it
// (uses *sh and barriers).
__device__ inline int stage_n_chunk(const PruneArgs &a, const Problem &pr, int p, int nthreads, int *sh)
{
    if (a.parent_starts == nullptr) return max(0, (pr.hi - pr.lo + a.chunk - 1) / a.chunk);
    if (threadIdx.x == 0) *sh = 0;
    __syncthreads();
    const int32_t *ps = a.parent_starts + (int64_t)p * a.n_parent;
    const int parent_chunk = a.chunk << a.ratio_log2;
    for (int i = threadIdx.x; i < a.n_parent; i += nthreads) {
        const int s0 = ps[i];
        const bool here = s0 >= 0 && s0 < pr.hi;
        const int s1 = i + 1 < a.n_parent ? ps[i + 1] : -1;
        if (here && !(s1 >= 0 && s1 < pr.hi))       // the last parent that holds keys
            *sh = (i << a.ratio_log2) + (min(parent_chunk, pr.hi - s0) + a.chunk - 1) / a.chunk;
    }
    __syncthreads();
    return *sh;
}

// SRC 0: K in HBM through strides; 1: host tier with the on-GPU bank; 2: paged pool
template <int SRC> struct KeySource;
template <> struct KeySource<0> {
    typedef DirectRows type;
    static __device__ type make(const PruneArgs &a, const Problem &pr)
    {
        return DirectRows{a.k + pr.b * a.k_sb + pr.g * a.k_sh, a.k_st};
    }
};
template <> struct KeySource<1> {
    typedef CachedRows type;
    static __device__ type make(const PruneArgs &a, const Problem &pr)
    {
        return cached_rows(a.bank, a.k, a.k_sb, a.k_sh, a.k_st, a.bank.bank_k, pr.b, pr.g, a.ge.Hkv);
    }
};

template <> struct KeySource<2> {
    typedef PagedRows type;
    static __device__ type make(const PruneArgs &a, const Problem &pr)
    {
        return PagedRows{a.k + pr.g * a.k_sh, a.paged.block_table + (int64_t)pr.b * a.paged.table_stride, a.k_sb,
                         a.k_st, a.paged.page_log2};
    }
};

}  // namespace ihip
