// The selections of several stages that were scored together (prune_decode_nest.h), in one launch: a workgroup per problem, or
// per set of pooled problems.
//
// A selection is a chain of short steps; as kernels of their own each also pays its launch, the way of its inputs from memory and
// its drain.  Here all scores of the problem are brought to LDS first, and every stage selects among the children of the
// chunks that the stage before it kept, whose scores are there already.
//
// One selection: the candidates' scores go into 512 linear bins, the K-th best lies in one of them, whose candidates are ranked
// exactly by (score descending, slot ascending).  Any range serves for the bins, since scores beyond it go into the outermost
// ones: it is that of 64 scores of the stage, and half as much again above (more is kept of low scores than of high ones), so
// that no pass over all of them and no exchange between the waves is needed for it.  512 bins are what a wave can sum by
// itself, and so are the few candidates of a bin, one to a lane: every wave finds the K-th best's bin and the last slot that is kept of it
// without a barrier.  Heavy ties (more candidates in that bin than lanes) go through the radix selection of block_select.h.  Two stages,
// 1,500 candidates of the first, as many equal ones in the bin (us), candidates ranked by their owners up to 512 / so: 1 11.2 / 9.7,
// 64 53 / 16, 65 56 / 20, 300 153 / 20, 700 25 / 23.  Four barriers a stage.  A wave's candidates lie together, item after item, so that ballots put the kept ones in order.
//
// What bounds it is a chain of latencies, of which code that runs for the first time is a part: instructions come from beyond the
// instruction cache, so a stage's code is short and the same for all stages.  Two stages of 2,048 candidates, 512 kept (us): candidates
// ranked by their owners, a loop for each item, scores fetched in three turns 14.2; this way 8.8; 256 candidates each 6.8 / 6.0.
#include "select_chain.h"

namespace ihip {

struct ChainArgs {
    Geometry ge;
    ChainPlan plan;
};

constexpr int kChainBins = 512;            // eight per lane
// One sequence of 8K keys, a layer (us): 512 threads 24.2, 256 24.8, 1024 26.4
constexpr int kChainThreads = 512;

template <bool PARENTS>
struct ChainShared {
    float score[kChainMaxScores];
    int32_t index[2][kChainMaxKeep];          // what a stage kept: slots in its score row, which is the middle range, or the parents' keys, in order
    alignas(16) uint32_t hist[kChainMaxStages][kChainBins];       // read four bins at a time
    uint2 cand[64];                           // key and slot
    uint32_t ncand[kChainMaxStages], total[kChainThreads / 64];
    SelectScratch<kChainThreads> scratch;
    int32_t parent[PARENTS ? kChainMaxParents : 1];
};

// Monotone map fp32 -> u32 (larger float <=> larger key); -0.0 maps with +0.0.
__device__ inline uint32_t chain_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Selects stage s of the chain from n candidates, children of the n_from chunks that the stage before it kept.  -> how many are kept
template <int ITEMS, class Shared>
__device__ inline int chain_stage(const ChainPlan &c, int s, int n, int n_from, const float *score, float low, float scale, Shared &sh)
{
    constexpr int NT = kChainThreads, kWaves = NT / 64;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int32_t *from_index = sh.index[(s & 1) ^ 1];
    int32_t *to_index = sh.index[s & 1];
    uint32_t *hist = sh.hist[s];
    const int ratio_log2 = c.ratio_log2[s], mask = (1 << ratio_log2) - 1;
    // candidate i: its slot in the score row
    auto slot_of = [&](int i) { return s > 0 ? (from_index[i >> ratio_log2] << ratio_log2) | (i & mask) : i; };
    const int limit = s > 0 ? min(n, n_from << ratio_log2) : n;
    const int i0 = wv * 64 * ITEMS + lane;    // a wave's candidates lie together, item k of all lanes after item k - 1
    float v[ITEMS];
    int b[ITEMS], slot[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) slot[k] = slot_of(i0 + 64 * k < limit ? i0 + 64 * k : 0);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) v[k] = i0 + 64 * k < limit ? score[slot[k]] : -INFINITY;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        b[k] = v[k] > -INFINITY ? max(0, min(kChainBins - 1, (int)((v[k] - low) * scale))) : -1;
        if (b[k] >= 0) atomicAdd(&hist[b[k]], 1u);
    }
    __syncthreads();
    // Every wave by itself: lane l sums the bins from 511 - 8 l down; of the eight in which the K-th best lies lanes 0..7 take one each
    uint32_t sum;
    {
        const uint4 *h4 = reinterpret_cast<const uint4 *>(&hist[kChainBins - 8 * (lane + 1)]);
        const uint4 x = h4[0], y = h4[1];
        sum = ((x.x + x.y) + (x.z + x.w)) + ((y.x + y.y) + (y.z + y.w));
    }
    const uint32_t upto = wave_scan_u32(sum, lane);
    const int keep = min(__builtin_amdgcn_readlane((int)upto, 63), c.keep[s]);
    if (keep > 0) {
        const int at = __ffsll((unsigned long long)__ballot(upto >= (uint32_t)keep)) - 1;
        const int top = kChainBins - 1 - 8 * at;
        const uint32_t h = lane < 8 ? hist[top - lane] : 0u;
        const uint32_t run = (uint32_t)__builtin_amdgcn_readlane((int)(upto - sum), at) + wave_scan_u32(h, lane);
        const int j = __ffsll((unsigned long long)__ballot(run >= (uint32_t)keep)) - 1;
        const int tb = top - j;
        const uint32_t n_cand = (uint32_t)__builtin_amdgcn_readlane((int)h, j);
        const uint32_t need = keep - ((uint32_t)__builtin_amdgcn_readlane((int)run, j) - n_cand);
        if (n_cand <= 64u) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k)
                if (b[k] == tb) sh.cand[atomicAdd(&sh.ncand[s], 1u)] = make_uint2(chain_key(v[k]), (uint32_t)slot[k]);
            __syncthreads();
            // every wave ranks them for itself, one a lane, and finds the last one kept
            const uint2 me = sh.cand[min((uint32_t)lane, n_cand - 1)];
            uint32_t rank = 0;
            for (uint32_t o = 0; o < n_cand; ++o) {
                const uint32_t okey = (uint32_t)__builtin_amdgcn_readlane((int)me.x, (int)o), oslot = (uint32_t)__builtin_amdgcn_readlane((int)me.y, (int)o);
                rank += okey > me.x || (okey == me.x && oslot < me.y);
            }
            const int last = __ffsll((unsigned long long)__ballot((uint32_t)lane < n_cand && rank == need - 1)) - 1;
            const uint32_t last_key = (uint32_t)__builtin_amdgcn_readlane((int)me.x, last);
            const int last_slot = __builtin_amdgcn_readlane((int)me.y, last);
            uint64_t m[ITEMS];
            int cnt = 0;
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const uint32_t key = chain_key(v[k]);
                m[k] = __ballot(b[k] > tb || (b[k] == tb && (key > last_key || (key == last_key && slot[k] <= last_slot))));
                cnt += __popcll(m[k]);
            }
            if (lane == 0) sh.total[wv] = cnt;
            __syncthreads();
            int pos = (int)wave_sum_u32(lane < wv ? sh.total[lane & (kWaves - 1)] : 0u);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                if ((m[k] >> lane) & 1) to_index[pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], 0u))] = slot[k];
                pos += __popcll(m[k]);
            }
        } else {
            block_select_largest<NT>(
                limit, keep, [&](int i) { return chain_key(score[slot_of(i)]); },
                [&](uint32_t rank, int i) { to_index[rank] = slot_of(i); }, sh.scratch);
        }
    }
    __syncthreads();
    return keep;
}

template <bool PARENTS>
__global__ __launch_bounds__(kChainThreads) void select_chain_kernel(const ChainArgs args, const ChainParents parents)
{
    constexpr int NT = kChainThreads;
    __shared__ __attribute__((aligned(16))) ChainShared<PARENTS> sh;
    const Geometry &ge = args.ge;
    const ChainPlan &c = args.plan;
    const int p0 = c.pool > 1 ? blockIdx.x * ge.Hkv : blockIdx.x;      // the first problem of a pooled set; decode: one block per sequence
    const int tid = threadIdx.x, lane = tid & 63;
    {
        // all scores are asked for at once (rows are whole 256 bytes)
        const float4 *row = reinterpret_cast<const float4 *>(c.scores + (int64_t)p0 * c.stride);
        const int n4 = c.stride >> 2;
        float4 *to = reinterpret_cast<float4 *>(sh.score);
        constexpr int kAhead = kChainMaxScores / 4 / NT;
        float4 x[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (k * NT < n4) x[k] = row[min(tid + k * NT, n4 - 1)];
        for (int i = tid; i < kChainMaxStages * kChainBins / 4; i += NT) reinterpret_cast<uint4 *>(sh.hist[0])[i] = make_uint4(0, 0, 0, 0);
        if (tid < kChainMaxStages) sh.ncand[tid] = 0u;
        if constexpr (PARENTS)
            for (int i = tid; i < parents.n; i += NT) sh.parent[i] = parents.starts[(int64_t)p0 * parents.n + i];
        // Pooled heads, seven at once: one trip to memory for each 2,048 scores of eight heads, where head after head is seven for each
        // 16,384.  Layers, head after head / so (us): 16 heads on 8, 15K bf16 keys in pages 34.1 / 28.8; 64 on 8, 5 of 20K E4M3 54.4 / 49.3
        for (int g = 1; g < c.pool; g += 7) {
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
                if (k * NT < n4) {
                    const float4 *others = row + min(tid + k * NT, n4 - 1);
                    float4 y[7];
#pragma unroll
                    for (int h = 0; h < 7; ++h) y[h] = others[(int64_t)min(g + h, c.pool - 1) * n4];
#pragma unroll
                    for (int h = 0; h < 7; ++h)
                        x[k] = make_float4(fmaxf(x[k].x, y[h].x), fmaxf(x[k].y, y[h].y), fmaxf(x[k].z, y[h].z), fmaxf(x[k].w, y[h].w));
                }
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k)          // -0.0 -> +0.0
            if (tid + k * NT < n4) to[tid + k * NT] = make_float4(x[k].x + 0.0f, x[k].y + 0.0f, x[k].z + 0.0f, x[k].w + 0.0f);
    }
    const Problem pr = problem_of(ge, p0);
    __syncthreads();
    int kept = 0;
    for (int s = 0; s < c.n_stages; ++s) {
        const int n = s == 0 ? c.slots[0] : c.keep[s - 1] << c.ratio_log2[s];
        const float *score = sh.score + c.at[s];
        // the bins, from 64 of the stage's scores (every wave for itself)
        const float x = score[(int)((uint32_t)lane * (uint32_t)c.slots[s] >> 6)];
        const float low = wave_min_f32(x > -INFINITY ? x : INFINITY), high = wave_max_f32(x);
        const float scale = high > low ? (float)kChainBins / (1.5f * (high - low)) : 0.f;
        if (n <= NT) kept = chain_stage<1>(c, s, n, kept, score, low, scale, sh);
        else kept = chain_stage<4>(c, s, n, kept, score, low, scale, sh);
        for (int g = 0; g < c.pool; ++g) {
            int32_t *out = c.out[s] + (int64_t)(p0 + g) * c.keep[s];
            for (int i = tid; i < c.keep[s]; i += NT) {
                if constexpr (PARENTS) {
                    const int f = i < kept ? sh.index[s & 1][i] * c.chunk[s] : 0;
                    out[i] = i < kept ? sh.parent[f >> parents.log2] + (f & ((1 << parents.log2) - 1)) : -1;
                } else {
                    out[i] = i < kept ? pr.lo + sh.index[s & 1][i] * c.chunk[s] : -1;
                }
            }
        }
    }
}

int32_t launch_select_chain(const ihip_shape &s, const ChainPlan &plan, const ChainParents &parents, hipStream_t st)
{
    const int P = s.B * (plan.pool > 1 ? 1 : s.Hkv);
    KernelTimer timer(stage_name(kNameSelect, parents.starts == nullptr, plan.chunk[0]), st);
    const ChainArgs args{make_geometry(s), plan};
    if (parents.starts != nullptr) hipLaunchKernelGGL(select_chain_kernel<true>, dim3(P), dim3(kChainThreads), 0, st, args, parents);
    else hipLaunchKernelGGL(select_chain_kernel<false>, dim3(P), dim3(kChainThreads), 0, st, args, parents);
    return check_launch("select_blocks (several stages)");
}

}  // namespace ihip
