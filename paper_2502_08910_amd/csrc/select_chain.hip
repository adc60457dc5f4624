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
// itself, so every wave finds the K-th best's bin without a barrier.  Heavy ties (more candidates in that bin than
// threads) go through the radix selection of block_select.h.  Four barriers a stage.
#include "select_chain.h"

namespace ihip {

struct ChainArgs {
    Geometry ge;
    ChainPlan plan;
};

constexpr int kChainBins = 512;            // eight per lane
// One sequence of 8K keys, a layer (us): 512 threads 24.2, 256 24.8, 1024 26.4
constexpr int kChainThreads = 512;

struct ChainShared {
    float score[kChainMaxScores];
    int32_t index[2][kChainMaxKeep];          // what a stage kept: slots in its score row, which is the middle range in order
    uint32_t hist[kChainMaxStages][kChainBins];
    uint2 cand[kChainThreads];                           // key and candidate
    uint32_t ncand[kChainMaxStages], total[kChainThreads / 64];
    SelectScratch<kChainThreads> scratch;
};

// Monotone map fp32 -> u32 (larger float <=> larger key); -0.0 maps with +0.0.
__device__ inline uint32_t chain_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Selects stage s of the chain from n candidates, children of the n_from chunks that the stage before it kept.  -> how many are kept
template <int ITEMS>
__device__ inline int chain_stage(const ChainPlan &c, int s, int n, int n_from, const float *score, float low, float scale, ChainShared &sh)
{
    constexpr int NT = kChainThreads, kWaves = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t *from_index = sh.index[(s & 1) ^ 1];
    int32_t *to_index = sh.index[s & 1];
    uint32_t *hist = sh.hist[s];
    const int ratio_log2 = c.ratio_log2[s], mask = (1 << ratio_log2) - 1;
    // candidate i: its slot in the score row
    auto slot_of = [&](int i) { return s > 0 ? (from_index[i >> ratio_log2] << ratio_log2) | (i & mask) : i; };
    const int limit = s > 0 ? min(n, n_from << ratio_log2) : n;
    const int i0 = tid * ITEMS;
    float v[ITEMS];
    int b[ITEMS], slot[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) slot[i] = slot_of(i0 + i < limit ? i0 + i : 0);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) v[i] = i0 + i < limit ? score[slot[i]] : -INFINITY;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        b[i] = v[i] > -INFINITY ? max(0, min(kChainBins - 1, (int)((v[i] - low) * scale))) : -1;
        if (b[i] >= 0) atomicAdd(&hist[b[i]], 1u);
    }
    __syncthreads();
    // Every wave by itself: lane l sums the bins from 511 - 8 l down
    uint32_t h[8], sum = 0;
    {
        const uint4 *h4 = reinterpret_cast<const uint4 *>(&hist[kChainBins - 8 * (lane + 1)]);
        const uint4 x = h4[0], y = h4[1];
        h[0] = y.w; h[1] = y.z; h[2] = y.y; h[3] = y.x; h[4] = x.w; h[5] = x.z; h[6] = x.y; h[7] = x.x;
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += h[j];
    }
    const uint32_t upto = wave_scan_u32(sum, lane);
    const int keep = min(__builtin_amdgcn_readlane((int)upto, 63), c.keep[s]);
    if (keep > 0) {
        const int at = __ffsll((unsigned long long)__ballot(upto >= (uint32_t)keep)) - 1;
        uint32_t run = upto - sum, above_l = 0, count_l = 0;
        int bin_l = -1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool here = bin_l < 0 && run + h[j] >= (uint32_t)keep;
            bin_l = here ? kChainBins - 1 - 8 * lane - j : bin_l;
            above_l = here ? run : above_l;
            count_l = here ? h[j] : count_l;
            run += h[j];
        }
        const int tb = __builtin_amdgcn_readlane(bin_l, at);
        const uint32_t need = keep - (uint32_t)__builtin_amdgcn_readlane((int)above_l, at), n_cand = (uint32_t)__builtin_amdgcn_readlane((int)count_l, at);
        if (n_cand <= (uint32_t)NT) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (b[i] == tb) {
                    const uint32_t at = atomicAdd(&sh.ncand[s], 1u);
                    sh.cand[at] = make_uint2(chain_key(v[i]), i0 + i);
                }
            __syncthreads();
            bool take[ITEMS];
            uint32_t cnt = 0;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                take[i] = b[i] > tb;
                if (b[i] == tb) {             // ranked among the bin's candidates by its owner
                    const uint32_t mk = chain_key(v[i]), me = i0 + i;
                    uint32_t rank = 0;
                    for (uint32_t j = 0; j < n_cand; j += 4) {
                        uint2 o[4];           // read together
#pragma unroll
                        for (int k = 0; k < 4; ++k) o[k] = sh.cand[min(j + k, (uint32_t)NT - 1)];
#pragma unroll
                        for (int k = 0; k < 4; ++k) rank += j + k < n_cand && (o[k].x > mk || (o[k].x == mk && o[k].y < me));
                    }
                    take[i] = rank < need;
                }
                cnt += take[i];
            }
            const uint32_t incl = wave_scan_u32(cnt, lane);
            if (lane == 63) sh.total[wv] = incl;
            __syncthreads();
            uint32_t pos = incl - cnt + wave_sum_u32(lane < wv ? sh.total[lane & (kWaves - 1)] : 0u);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (take[i]) to_index[pos++] = slot[i];
        } else {
            block_select_largest<NT>(
                limit, keep, [&](int i) { return chain_key(score[slot_of(i)]); },
                [&](uint32_t rank, int i) { to_index[rank] = slot_of(i); }, sh.scratch);
        }
    }
    __syncthreads();
    return keep;
}

__global__ __launch_bounds__(kChainThreads) void select_chain_kernel(const ChainArgs args)
{
    constexpr int NT = kChainThreads;
    __shared__ ChainShared sh;
    const Geometry &ge = args.ge;
    const ChainPlan &c = args.plan;
    const int p0 = c.pool > 1 ? blockIdx.x * ge.Hkv : blockIdx.x;      // the first problem of a pooled set; decode: one block per sequence
    const int tid = threadIdx.x, lane = tid & 63;
    const Problem pr = problem_of(ge, p0);
    for (int i = tid; i < kChainMaxStages * kChainBins / 4; i += NT) reinterpret_cast<uint4 *>(sh.hist[0])[i] = make_uint4(0, 0, 0, 0);
    if (tid < kChainMaxStages) sh.ncand[tid] = 0u;
    {
        const float *row = c.scores + (int64_t)p0 * c.stride;
        constexpr int kAhead = 8;
        for (int i0 = tid; i0 < c.stride; i0 += kAhead * NT) {
            float x[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) x[k] = row[min(i0 + k * NT, c.stride - 1)];
            for (int g = 1; g < c.pool; ++g)
#pragma unroll
                for (int k = 0; k < kAhead; ++k) x[k] = fmaxf(x[k], row[(int64_t)g * c.stride + min(i0 + k * NT, c.stride - 1)]);
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
                if (i0 + k * NT < c.stride) sh.score[i0 + k * NT] = x[k] + 0.0f;                  // -0.0 -> +0.0
        }
    }
    __syncthreads();
    // the bins of every stage, from 64 of its scores (every wave for itself)
    float low[kChainMaxStages], scale[kChainMaxStages];
#pragma unroll
    for (int s = 0; s < kChainMaxStages; ++s) {
        const int of = s < c.n_stages ? s : 0;           // without a branch, so that the stages' steps interleave
        const float x = sh.score[c.at[of] + (int)((uint32_t)lane * (uint32_t)c.slots[of] >> 6)];
        const float mn = wave_min_f32(x > -INFINITY ? x : INFINITY), mx = wave_max_f32(x);
        low[s] = mn;
        scale[s] = mx > mn ? (float)kChainBins / (1.5f * (mx - mn)) : 0.f;
    }
    int kept = 0;
    for (int s = 0; s < c.n_stages; ++s) {
        const int n = s == 0 ? c.slots[0] : c.keep[s - 1] << c.ratio_log2[s];
        const float *score = sh.score + c.at[s];
        const float lo = s == 0 ? low[0] : s == 1 ? low[1] : s == 2 ? low[2] : low[3];
        const float sc = s == 0 ? scale[0] : s == 1 ? scale[1] : s == 2 ? scale[2] : scale[3];
        if (n <= NT) kept = chain_stage<1>(c, s, n, kept, score, lo, sc, sh);
        else if (n <= 2 * NT) kept = chain_stage<2>(c, s, n, kept, score, lo, sc, sh);
        else kept = chain_stage<4>(c, s, n, kept, score, lo, sc, sh);
        for (int g = 0; g < c.pool; ++g) {
            int32_t *out = c.out[s] + (int64_t)(p0 + g) * c.keep[s];
            for (int i = tid; i < c.keep[s]; i += NT) out[i] = i < kept ? pr.lo + sh.index[s & 1][i] * c.chunk[s] : -1;
        }
    }
}

int32_t launch_select_chain(const ihip_shape &s, const ChainPlan &plan, hipStream_t st)
{
    const int P = s.B * (plan.pool > 1 ? 1 : s.Hkv);
    KernelTimer timer(stage_name(kNameSelect, true, plan.chunk[0]), st);
    const ChainArgs args{make_geometry(s), plan};
    hipLaunchKernelGGL(select_chain_kernel, dim3(P), dim3(kChainThreads), 0, st, args);
    return check_launch("select_blocks (several stages)");
}

}  // namespace ihip
