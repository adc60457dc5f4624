// The selections of several stages that were scored together (prune_decode_nest.h), in one launch: a workgroup per problem, or
// per set of pooled problems.
//
// A selection is a chain of short steps; as kernels of their own each also pays its launch, the way of its inputs from memory and
// its drain.  Here all scores of the problem are brought to LDS first, and every stage selects among the children of the
// chunks that the stage before it kept, whose scores are there already.  1,024 threads: with two to four candidates a
// thread its steps are a few instructions each.
//
// One selection: scores into 2,048 linear bins between the smallest and the largest, the K-th best lies in one of them, its
// candidates are ranked exactly by (score descending, slot ascending).  Heavy ties (more candidates in that bin than
// threads) go through the radix selection of block_select.h.
#include "select_chain.h"
#include <algorithm>

namespace ihip {

struct ChainArgs {
    Geometry ge;
    ChainPlan plan;
};

constexpr int kChainBins = 2048;

template <int NT>
struct ChainShared {
    float score[kChainMaxScores];
    int32_t index[2][kChainMaxKeep], start[2][kChainMaxKeep];      // what the stages kept: slot in the stage's score row, first key
    uint32_t hist[kChainBins];
    uint32_t cand[NT], cand_key[NT];
    float lo[NT / 64], hi[NT / 64];
    uint32_t count[NT / 64], total[NT / 64];
    uint32_t segment[16];
    uint32_t ncand;
    SelectScratch<NT> scratch;
};

// Monotone map fp32 -> u32 (larger float <=> larger key); -0.0 maps with +0.0.
__device__ inline uint32_t chain_key(float f)
{
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Selects stage s of the chain from n candidates; kept_before: how many the stage before kept.  -> how many are kept
template <int NT, int ITEMS>
__device__ inline int chain_stage(const Geometry &ge, const ChainPlan &c, int s, int n, int kept_before, const Problem &pr, int p0, const float *score,
                                  ChainShared<NT> &sh)
{
    constexpr int kWaves = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t *from_index = sh.index[(s & 1) ^ 1], *from_start = sh.start[(s & 1) ^ 1];
    int32_t *to_index = sh.index[s & 1], *to_start = sh.start[s & 1];
    const int ratio_log2 = c.ratio_log2[s], chunk = c.chunk[s];
    // candidate i: its slot in the score row and its first key
    auto slot_of = [&](int i) { return s == 0 ? i : (from_index[i >> ratio_log2] << ratio_log2) | (i & ((1 << ratio_log2) - 1)); };
    auto start_of = [&](int i) {
        if (s == 0) return slot_start(pr, c.parent_starts, c.n_parent, ratio_log2, chunk, p0, i);
        return from_start[i >> ratio_log2] + (i & ((1 << ratio_log2) - 1)) * chunk;
    };
    const int limit = s == 0 ? n : min(n, kept_before << ratio_log2);
    float v[ITEMS];
    const int i0 = tid * ITEMS;
    float mn = INFINITY, mx = -INFINITY;
    uint32_t valid = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        v[i] = i0 + i < limit ? score[slot_of(i0 + i)] + 0.0f : -INFINITY;          // -0.0 -> +0.0
        const bool there = v[i] > -INFINITY;
        mn = there ? fminf(mn, v[i]) : mn;
        mx = fmaxf(mx, v[i]);
        valid += __popcll(__ballot(there));
    }
    mn = wave_min_f32(mn);
    mx = wave_max_f32(mx);
    if (lane == 0) { sh.lo[wv] = mn; sh.hi[wv] = mx; sh.count[wv] = valid; }
#pragma unroll
    for (int i = 0; i < kChainBins / NT; ++i) sh.hist[tid + i * NT] = 0;
    if (tid == 0) sh.ncand = 0;
    __syncthreads();
    // every wave reduces the waves' values itself
    {
        const int w = lane & (kWaves - 1);
        mn = wave_min_f32(sh.lo[w]);
        mx = wave_max_f32(sh.hi[w]);
        valid = wave_sum_u32(lane < kWaves ? sh.count[w] : 0u);
    }
    const int keep = min((int)valid, c.keep[s]);
    if (keep > 0) {
        const float scale = mx > mn ? (float)(kChainBins - 1) / (mx - mn) : 0.f;
        int b[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            b[i] = v[i] > -INFINITY ? min(kChainBins - 1, (int)((v[i] - mn) * scale)) : -1;
            if (b[i] >= 0) atomicAdd(&sh.hist[b[i]], 1u);
        }
        __syncthreads();
        // Sixteen segments of 128 bins, the highest first, are summed by the waves; then every wave finds for itself the segment,
        // and in it the bin, where the count from the top reaches `keep`.
        constexpr int kSegments = 16, kSeg = kChainBins / kSegments;
        auto segment = [&](int w) { return *reinterpret_cast<const uint2 *>(&sh.hist[kChainBins - kSeg * w - 2 * lane - 2]); };
#pragma unroll
        for (int w = 0; w < kSegments / kWaves; ++w) {
            const uint2 h = segment(w * kWaves + wv);
            const uint32_t sum = wave_sum_u32(h.x + h.y);
            if (lane == 0) sh.segment[w * kWaves + wv] = sum;
        }
        __syncthreads();
        int tb;
        uint32_t above;
        {
            const uint32_t t = lane < kSegments ? sh.segment[lane & (kSegments - 1)] : 0u;
            const uint32_t upto = wave_scan_u32(t, lane);
            const int seg = __ffsll((unsigned long long)__ballot(upto >= (uint32_t)keep)) - 1;
            const uint2 h = segment(seg);
            const uint32_t run = wave_scan_u32(h.x + h.y, lane) + (uint32_t)__builtin_amdgcn_readlane((int)(upto - t), seg);
            const int at = __ffsll((unsigned long long)__ballot(run >= (uint32_t)keep)) - 1;
            const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(run - h.x - h.y), at), high = (uint32_t)__builtin_amdgcn_readlane((int)h.y, at);
            const bool in_high = before + high >= (uint32_t)keep;
            tb = kChainBins - 1 - kSeg * seg - 2 * at - (in_high ? 0 : 1);
            above = in_high ? before : before + high;
        }
        const uint32_t need = keep - above, n_cand = sh.hist[tb];
        if (n_cand <= (uint32_t)NT) {
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                if (b[i] == tb) {
                    const uint32_t at = atomicAdd(&sh.ncand, 1u);
                    sh.cand[at] = i0 + i;
                    sh.cand_key[at] = chain_key(v[i]);
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
                    for (uint32_t j = 0; j < n_cand; ++j) {
                        const uint32_t o = sh.cand[j], ok = sh.cand_key[j];
                        rank += (ok > mk) || (ok == mk && o < me);
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
                if (take[i]) {
                    to_index[pos] = slot_of(i0 + i);
                    to_start[pos] = start_of(i0 + i);
                    ++pos;
                }
        } else {
            block_select_largest<NT>(
                limit, keep, [&](int i) { return chain_key(score[slot_of(i)]); },
                [&](uint32_t rank, int i) { to_index[rank] = slot_of(i); to_start[rank] = start_of(i); }, sh.scratch);
        }
    }
    __syncthreads();
    return keep;
}

template <int NT>
__global__ __launch_bounds__(NT) void select_chain_kernel(const ChainArgs args)
{
    __shared__ ChainShared<NT> sh;
    const Geometry &ge = args.ge;
    const ChainPlan &c = args.plan;
    const int p0 = c.pool > 1 ? blockIdx.x * ge.Hkv : blockIdx.x;      // the first problem of a pooled set; decode: one block per sequence
    const Problem pr = problem_of(ge, p0);
    const int tid = threadIdx.x;
    // all scores, rows of pooled heads c.stride apart
    {
        const float *row = c.scores + (int64_t)p0 * c.stride;
        const int n = c.stride;
        for (int i = tid; i < n; i += 8 * NT) {
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = row[min(i + k * NT, n - 1)];
            for (int g = 1; g < c.pool; ++g)
#pragma unroll
                for (int k = 0; k < 8; ++k) x[k] = fmaxf(x[k], row[(int64_t)g * n + min(i + k * NT, n - 1)]);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i + k * NT < n) sh.score[i + k * NT] = x[k];
        }
    }
    __syncthreads();
    int kept = 0;
    const float *score = sh.score;
    for (int s = 0; s < c.n_stages; ++s) {
        const int n = s == 0 ? c.slots[0] : c.keep[s - 1] << c.ratio_log2[s];
        if (n <= NT) kept = chain_stage<NT, 1>(ge, c, s, n, kept, pr, p0, score, sh);
        else if (n <= 2 * NT) kept = chain_stage<NT, 2>(ge, c, s, n, kept, pr, p0, score, sh);
        else kept = chain_stage<NT, 4>(ge, c, s, n, kept, pr, p0, score, sh);
        score += c.slots[s];
        for (int g = 0; g < c.pool; ++g) {
            int32_t *out = c.out[s] + (int64_t)(p0 + g) * c.keep[s];
            for (int i = tid; i < c.keep[s]; i += NT) out[i] = i < kept ? sh.start[s & 1][i] : -1;
        }
    }
}

int32_t launch_select_chain(const ihip_shape &s, const ChainPlan &plan, hipStream_t st)
{
    const int P = s.B * (plan.pool > 1 ? 1 : s.Hkv);
    KernelTimer timer(stage_name(kNameSelect, plan.parent_starts == nullptr, plan.chunk[0]), st);
    int most = plan.slots[0];
    for (int i = 1; i < plan.n_stages; ++i) most = std::max(most, plan.keep[i - 1] << plan.ratio_log2[i]);
    const ChainArgs args{make_geometry(s), plan};
    if (most <= 512) hipLaunchKernelGGL(select_chain_kernel<256>, dim3(P), dim3(256), 0, st, args);
    else if (most <= 1024) hipLaunchKernelGGL(select_chain_kernel<512>, dim3(P), dim3(512), 0, st, args);
    else hipLaunchKernelGGL(select_chain_kernel<1024>, dim3(P), dim3(1024), 0, st, args);
    return check_launch("select_blocks (several stages)");
}

}  // namespace ihip
