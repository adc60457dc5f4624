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

// The grid of a decode stage's launch.  Where the heads of a token lie beside each other (token-major rows, pages) problems dealt out
// first read the same few rows of memory at once from all XCDs, and over pages a ragged batch also ends with a few long sequences
// whose pages are all still to be looked up: there the part stays fastest on long contexts.  Layers, 8 KV heads, part / problem
// fastest (us, second pair ragged):
//   bf16 pages, and token-major bf16 rows without RoPE, by the keys of all sequences, line 768K: pages, 4 sequences of 64K 64.2 / 61.7 and
//     65.4 / 62.1, 16 of 32K 129.2 / 129.4 and 126.1 / 126.8, 4 of 250K 111.5 / 112.0 and 104.8 / 108.3, 8 of 500K 302 / 301 and
//     268 / 280; rows, 4 of 64K 61.1 / 57.6, 4 of 250K 110.8 / 108.7 and 100.5 / 101.9, one of 1M 96.2 / 103.9, 8 of 500K 287 / 310 and 264 / 287
//   token-major rows with RoPE, by the keys of a sequence, line 288K for E4M3 and 384K for bf16: E4M3, 16 of 128K 288.7 / 294.6, 12 of
//     333K 290 / 301 and 285 / 294, 8 of 500K 224 / 243 and 219 / 235; bf16, 16 of 128K 269.0 / 240.0, 12 of 333K 348 / 331 and
//     328 / 316, 8 of 500K 312 / 313 and 291 / 298, one of 1M 107 / 115
// E4M3 pages (8 of 500K with RoPE 237 / 236 and 221 / 222), token-major E4M3 without RoPE (198.6 / 180.1) and rows of a head in a row
// (303 / 297 and 277 / 276; RoPE 315.6 / 292.8) have no such loss.  Compare with buffers that lie alike: where a process's memory
// falls moves the largest of these by 3 %.
inline DecodeGrid prune_grid(const PruneArgs &a, int P, int per_problem, bool fp8, bool rope)
{
    const bool paged = a.paged.block_table != nullptr, token_major = !paged && std::abs(a.k_st) > std::abs(a.k_sh);
    const int64_t each = (int64_t)a.max_chunks * a.chunk, all = P / a.ge.Hkv * each;
    bool parts_first = a.bank.page_table != nullptr;
    if (paged || (token_major && !rope)) parts_first |= !fp8 && all > (int64_t)3 << 18;
    else if (token_major) parts_first |= each > (fp8 ? (int64_t)9 << 15 : (int64_t)3 << 17);
    return decode_grid(a.ge, per_problem, parts_first);
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
