// Block-sparse decode attention over sink + kept blocks + window.
//
// HBM-bound gather of K and V rows (512 B per attended token, shared by the G query heads of the KV head).  Flash-decoding layout: the
// attended tokens of a problem form a virtual slot list  [sink | kept blocks | window];  the list is cut into splits, one workgroup
// each; a wave takes 16 slots at a time, and every 16-lane row group reads four of their rows whole (16 B of a bf16 row per lane).
// The slots are dealt to the row groups in turn: token 4 * kq + u of the sixteen is slot 4 * u + kq, so that one load of the wave
// brings the rows of neighbouring slots.  HBM does not care, but over the host link 128-byte rows that a load names apart are
// requests of their own: host tier, 3,200 slots of 8 heads, nothing resident (us), four neighbouring slots to a row group / in turn:
// E4M3 149 / 120, with RoPE 165 / 120; bf16 239 / 237.
//
// On the vector ALUs a token costs some 26 instructions per 16 lanes and head -- dot, row reduction, a softmax that all lanes
// repeat, and 8 multiply-adds per head --, which was more than the rows' time with E4M3 rows, rotations or 8 heads.  The products are done
// on the matrix cores instead, in layouts between which no value crosses lanes:
//   scores   16 K rows x 16 columns (four v_mfma_f32_16x16x32_bf16; column n is head n % 4): lane (n, kq) gets its head's scores of
//            tokens 4 * kq .. + 3, the very tokens whose V rows its row group holds.  K goes to operand layout through LDS.
//   softmax  four scores a lane; the reference of the exponentials, and the sum, are the row group's own
//   output   v_mfma_f32_4x4x4_16B_bf16: 16 blocks of 4 heads x 4 tokens x 4 dims; a lane's four probabilities are its row of
//            the left operand, its 8 dims of the four V rows, in pairs of tokens, the columns of eight right ones.  A probability
//            goes in as three bf16 parts (24 bits), so nothing of it is rounded away (with finite V: the later parts are of
//            either sign or zero, and an infinite V gives NaN).
// With RoPE the keys are turned in fp32 and would need three parts as well (tried: 56 -> 63 us with four heads, 20 -> 29 with one), so
// their scores stay on the vector ALUs.  Split and merge, before / now (us): four heads, 16 sequences of 3,200 slots, bf16 45.8 / 38.9
// (5.4 TB/s), in pages 46.3 / 40.6, E4M3 38.4 / 26.3, bf16 with RoPE 56.4 / 43.5; 8 heads 75.6 / 41.4, 72.2 / 31.0, 96.9 / 52.3; one
// head 39.0 / 38.1; 4 sequences of 5,248 slots bf16 25.8 / 22.5, E4M3 24.4 / 16.9, bf16 with RoPE 33.1 / 27.1; one of 1,664 9.9 / 8.8.
// The rows of the next 16 slots are requested as soon as the registers of these are free (K once it is in LDS, V once it is
// in the products); a whole second set of registers leaves two waves per SIMD instead of four.
//
// Row groups and waves are merged at the end through row swaps and LDS, splits by a second small kernel (log-sum-exp merge).
#include "prune_decode_tile.h"
#include <algorithm>
#include <type_traits>

namespace ihip {

constexpr int kAttnThreads = 256;
constexpr int kAttnMaxSplit = 1536, kAttnUsualSplit = 1024;     // most slots of one split (multiples of 16); see decode_splits
constexpr int kAttnSplitCost = 128;                      // what beginning and ending a split costs, in slots; see decode_splits
constexpr int kAttnMinSplit = 256, kAttnMinSplitFine = 64;      // fewest; see decode_splits
// Log2 units that the reference of the exponentials is set above the scores that outgrew it, so that it seldom has to follow.  A
// probability is at most 1 then: sums of V rows overflow no sooner than with the maximum itself as the reference.
constexpr float kSlack = 8.f;
constexpr float kNegBig = -1.0e30f;                      // finite stand-in for -inf in running maxima

struct AttnDecodeArgs {
    Geometry ge;
    const uint16_t *q; int64_t q_sb, q_sh, q_st;
    const uint16_t *k; int64_t k_sb, k_sh, k_st;
    const uint16_t *v; int64_t v_sb, v_sh, v_st;
    const int32_t *block_starts;
    int n_blocks, block, block_log2;
    float scale_log2e;
    int n_splits, slots_per_split;
    DecodeGrid grid;
    float *part_ml;      // [P, n_splits, G, 2]   (running max in log2 units, sum)
    float *part_acc;     // [P, n_splits, G, 128]
    uint16_t *out;       // bf16 [B, Hq, 1, d]
    float *out_lse;      // [B, Hq] or null
    BankView bank;       // used by the cached instantiations only (K/V then point to host memory)
    const float *rope_cos, *rope_sin;   // streaming-style RoPE instantiations only: fp32 [n_pos][d/2]
    PagedView paged;     // paged instantiations only: K and V are page pools, *_sb the page strides
    float v_scale;       // FP8 instantiations: the output is multiplied by it (the K scale is folded into
                         // scale_log2e; K/V strides then count 2-byte units of the byte rows)
};

// SRC 0: K/V in HBM through strides; 1: host tier with the on-GPU bank; 2: paged pools
template <int SRC> struct KvSource;
template <> struct KvSource<0> {
    typedef DirectRows type;
    static __device__ type k(const AttnDecodeArgs &a, const Problem &pr)
    {
        return DirectRows{a.k + pr.b * a.k_sb + pr.g * a.k_sh, a.k_st};
    }
    static __device__ type v(const AttnDecodeArgs &a, const Problem &pr)
    {
        return DirectRows{a.v + pr.b * a.v_sb + pr.g * a.v_sh, a.v_st};
    }
};
template <> struct KvSource<1> {
    typedef CachedRows type;
    static __device__ type k(const AttnDecodeArgs &a, const Problem &pr)
    {
        return cached_rows(a.bank, a.k, a.k_sb, a.k_sh, a.k_st, a.bank.bank_k, pr.b, pr.g, a.ge.Hkv);
    }
    static __device__ type v(const AttnDecodeArgs &a, const Problem &pr)
    {
        return cached_rows(a.bank, a.v, a.v_sb, a.v_sh, a.v_st, a.bank.bank_v, pr.b, pr.g, a.ge.Hkv);
    }
};

template <> struct KvSource<2> {
    typedef PagedRows type;
    static __device__ type k(const AttnDecodeArgs &a, const Problem &pr)
    {
        return PagedRows{a.k + pr.g * a.k_sh, a.paged.block_table + (int64_t)pr.b * a.paged.table_stride, a.k_sb,
                         a.k_st, a.paged.page_log2};
    }
    static __device__ type v(const AttnDecodeArgs &a, const Problem &pr)
    {
        return PagedRows{a.v + pr.g * a.v_sh, a.paged.block_table + (int64_t)pr.b * a.paged.table_stride, a.v_sb,
                         a.v_st, a.paged.page_log2};
    }
};

typedef short bf16x4 __attribute__((ext_vector_type(4)));

// 8 dims turned, fp32
__device__ inline void turn8(float (&x)[8], const float4 c, const float4 sn)
{
    const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float e = x[2 * i], o = x[2 * i + 1];
        x[2 * i] = e * cc[i] - o * ss[i];
        x[2 * i + 1] = e * ss[i] + o * cc[i];
    }
}
// Sums over the 16 lanes of a row, of G values: lane n gets that of value n % 4 % G.  A step halves the values that a lane holds where
// there are any to halve: 44 instructions for the four heads of four tokens, 64 and a choice among the heads otherwise.
template <int G>
__device__ inline float head_sum(const float (&d)[G], int n)
{
    float x;
    if constexpr (G == 1) {
        x = d[0] + dpp_f32<0xB1>(d[0]);       // quad_perm [1,0,3,2]
        x += dpp_f32<0x4E>(x);                // quad_perm [2,3,0,1]
    } else {
        const bool odd = n & 1, high = n & 2;
        x = (odd ? d[1] : d[0]) + dpp_f32<0xB1>(odd ? d[0] : d[1]);
        if constexpr (G == 4) {
            const float y = (odd ? d[3] : d[2]) + dpp_f32<0xB1>(odd ? d[2] : d[3]);
            x = (high ? y : x) + dpp_f32<0x4E>(high ? x : y);
        } else {
            x += dpp_f32<0x4E>(x);
        }
    }
    x += dpp_f32<0x128>(x);                   // row_ror:8
    return x + dpp_f32<0x124>(x);             // row_ror:4
}

// Where the slot i of a split stands among its wave's tokens: 4 * kq + u for slot 4 * u + kq of sixteen
__device__ inline int slot_place(int i) { return (i & ~15) | ((i & 3) << 2) | ((i >> 2) & 3); }

// slot -> key position, or -1
__device__ inline int slot_to_pos(const AttnDecodeArgs &a, const Problem &pr, int p, int slot,
                                  int n_sink_eff, int w0)
{
    if (slot < n_sink_eff) return slot;
    slot -= n_sink_eff;
    const int nb = a.n_blocks << a.block_log2;
    if (slot < nb) {
        const int bs = a.block_starts[(int64_t)p * a.n_blocks + (slot >> a.block_log2)];
        if (bs < 0) return -1;
        const int pos = bs + (slot & (a.block - 1));
        return pos < pr.hi ? pos : -1;
    }
    const int pos = w0 + (slot - nb);
    return pos < pr.E ? pos : -1;
}

// ROPE: streaming-style positions (Sec. 4 "Dynamic RoPE ..."): the attended keys, in position
// order, are rotated to positions 0, 1, ..., n-1 and the query to n-1.  Attended slots are a
// prefix of the block part of the slot list (blocks are ascending, empty ones last, only the last
// one can be cut short), so a key's id is its slot, less the empty block slots for window keys.
// KV8: K and V rows are 128 bytes of E4M3, widened exactly to bf16.
template <int G, int SRC, bool ROPE, bool KV8>
__global__ __launch_bounds__(kAttnThreads, G == 8 ? 2 : ROPE && !(KV8 && G <= 2) ? 3 : 4) void attn_decode_split_kernel(const AttnDecodeArgs a)
{
    constexpr int NW = kAttnThreads / kWave;
    constexpr int kSets = G == 8 ? 2 : 1;                                   // of four heads (fewer: the four rows of a product repeat them)
    constexpr int kLoads = KV8 ? 2 : 4, kPieces = KV8 ? 8 : 16;             // of a lane for 16 K rows; 16-byte pieces of a row
    using v_t = typename std::conditional<KV8, uint2, uint4>::type;         // a lane's 8 dims of a V row
    const int p = a.grid.problem(), split = a.grid.part();
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const int s0 = split * a.slots_per_split;
    const int block_slots = a.n_blocks << a.block_log2;
    const int32_t *starts = a.block_starts + (int64_t)p * a.n_blocks;

    // The blocks of this thread's slots (of a split of the usual size) are asked for at once, next to the sequence's length, with the
    // whole sink there (which only a sequence shorter than it has not).
    constexpr int kSlots = kAttnUsualSplit / kAttnThreads;
    int start_of[kSlots];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
        const int i = tid + k * kAttnThreads, at = s0 + i - a.ge.n_sink;
        start_of[k] = i < a.slots_per_split && at >= 0 && at < block_slots ? starts[at >> a.block_log2] : -1;
    }
    const Problem pr = problem_of(a.ge, p);
    const int n_sink_eff = min(a.ge.n_sink, pr.E);
    const int w0 = max(pr.hi, a.ge.n_sink);

    __shared__ __attribute__((aligned(16))) int sh_pos[kAttnMaxSplit];      // key position of every slot of this split, at slot_place, -1 without one
    __shared__ __attribute__((aligned(16))) int sh_page[SRC == 2 ? kAttnMaxSplit : 4];       // paged K/V: the slot's page id
    __shared__ uint4 sh_rows[ROPE ? 1 : NW * 16 * kPieces];                 // 16 K rows of each wave on their way to operand layout
    __shared__ int sh_block_tokens;
    __shared__ __attribute__((aligned(16))) int sh_any[NW];                 // does a wave's share of the slots hold a key?
    const typename KvSource<SRC>::type ksrc = KvSource<SRC>::k(a, pr);
    const typename KvSource<SRC>::type vsrc = KvSource<SRC>::v(a, pr);
    // The queries, asked for now: column n's head of each set as an operand (head n % 4, n % G with fewer), or (ROPE) this lane's 8
    // dims of every head
    bf16x8 q[ROPE ? 1 : kSets][1][4];
    uint4 q_raw[ROPE ? G : 1];
    if constexpr (ROPE) {
#pragma unroll
        for (int h = 0; h < G; ++h) q_raw[h] = load_row16(a.q + pr.b * a.q_sb + (int64_t)(pr.g * G + h) * a.q_sh, 0, n);
    } else {
#pragma unroll
        for (int s = 0; s < kSets; ++s)
            decode_query_operands<KV8, 1>(a.q + pr.b * a.q_sb + (int64_t)(pr.g * G + s * 4 + (n & 3) % G) * a.q_sh, kq, RopeView{}, 0, q[s]);
    }
    int block_tokens = 0;
    if constexpr (ROPE) {
        // tokens in the kept blocks, so that window keys and the query know their ids
        if (tid == 0) sh_block_tokens = 0;
        __syncthreads();
        int mine = 0;
        for (int i0 = 0; i0 < a.n_blocks; i0 += 4 * kAttnThreads) {
            int bs[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) bs[k] = i0 + k * kAttnThreads + tid < a.n_blocks ? starts[i0 + k * kAttnThreads + tid] : -1;
#pragma unroll
            for (int k = 0; k < 4; ++k) mine += bs[k] >= 0 && bs[k] < pr.hi ? min(a.block, pr.hi - bs[k]) : 0;
        }
        mine = (int)wave_sum_u32((uint32_t)mine);
        if (lane == 0 && mine > 0) atomicAdd(&sh_block_tokens, mine);
    }
    bool any = false;
    auto put = [&](int i, int pos) {
        any |= pos >= 0;
        sh_pos[slot_place(i)] = pos;
        if constexpr (SRC == 2) sh_page[slot_place(i)] = pos >= 0 ? ksrc.table_entry(pos) : 0;
    };
#pragma unroll
    for (int k = 0; k < kSlots; ++k) {
        const int i = tid + k * kAttnThreads;
        if (i >= a.slots_per_split) break;
        int slot = s0 + i, pos;
        if (n_sink_eff == a.ge.n_sink) {
            const int at = slot - n_sink_eff;
            if (at < 0) pos = slot;
            else if (at < block_slots) {
                pos = start_of[k] + (at & (a.block - 1));
                pos = start_of[k] >= 0 && pos < pr.hi ? pos : -1;
            } else {
                pos = w0 + (at - block_slots);
                pos = pos < pr.E ? pos : -1;
            }
        } else {
            pos = slot_to_pos(a, pr, p, slot, n_sink_eff, w0);
        }
        put(i, pos);
    }
    for (int i = tid + kAttnUsualSplit; i < a.slots_per_split; i += kAttnThreads) put(i, slot_to_pos(a, pr, p, s0 + i, n_sink_eff, w0));
    const bool look = a.slots_per_split >= kAttnMinSplit;
    if (look) {
        any = __ballot(any) != 0;
        if (lane == 0) sh_any[wv] = any;
    }
    __syncthreads();
    const int64_t pbase = ((int64_t)p * a.n_splits + split) * G;
    // A split of absent blocks, as a plan for longer sequences has many: nothing to wait for (fine splits, which all run at once,
    // are not looked at).  One head a group, splits without keys walked / left (us): 27 sequences of 6,000 keys with 9,152 slots, bf16 115 / 111,
    // E4M3 77 / 61; layers of 7 sequences of 355 keys with 16,640 slots, bf16 24.4 / 21.9, E4M3 24.4 / 21.0
    if (look && (sh_any[0] | sh_any[1] | sh_any[2] | sh_any[3]) == 0) {
        for (int idx = tid; idx < G * kD; idx += kAttnThreads) a.part_acc[pbase * kD + idx] = 0.f;
        if (tid < 2 * G) a.part_ml[pbase * 2 + tid] = (tid & 1) ? 0.f : kNegBig;
        return;
    }

    f32x4 acc[kSets][8];                      // [dim of this lane's 8][head of the set]: of this row group's tokens
    float m[kSets], l[kSets];                 // of this row group's tokens, head n % 4: reference of the exponentials (log2 units), sum
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
        m[s] = kNegBig; l[s] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // 16 slots at a time, a wave's own.  Row group kq reads the K and V rows of tokens 4 * kq .. + 3, slots kq, 4 + kq, 8 + kq and 12 + kq.
    uint4 *stage = &sh_rows[wv * 16 * kPieces];
    uint4 kr[ROPE ? 1 : kLoads];
    v_t kv[ROPE ? 4 : 1], vr[4];              // ROPE: K rows as V rows, and their turns
    float4 tc[ROPE ? 4 : 1], ts[ROPE ? 4 : 1];
    auto four = [&](const int *of, int tile, int (&x)[4]) {
        const int4 w = *reinterpret_cast<const int4 *>(&of[tile * 16 + kq * 4]);
        x[0] = w.x; x[1] = w.y; x[2] = w.z; x[3] = w.w;
    };
    // id of the key of a slot: the slot, less the empty block slots if it is a window key
    auto key_id = [&](int slot, int pos) { return pos < 0 ? 0 : slot < n_sink_eff + block_slots ? slot : slot - (block_slots - block_tokens); };
    auto load_k = [&](int tile) {
        int pos[4], page[4] = {0, 0, 0, 0};
        four(sh_pos, tile, pos);
        if constexpr (SRC == 2) four(sh_page, tile, page);
        if constexpr (ROPE) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                kv[u] = v_t{};
                if (pos[u] >= 0) {
                    if constexpr (SRC == 2) kv[u] = *reinterpret_cast<const v_t *>(ksrc.row_in_page(page[u], pos[u]) + n * (KV8 ? 4 : 8));
                    else kv[u] = *reinterpret_cast<const v_t *>(ksrc.row(pos[u], n == 0) + n * (KV8 ? 4 : 8));
                }
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const bool second = KV8 && n >= 8;                  // E4M3: two rows of 8 lanes each
            const int at = KV8 ? (second ? pos[2 * i + 1] : pos[2 * i]) : pos[i];
            const int pg = KV8 ? (second ? page[2 * i + 1] : page[2 * i]) : page[i];
            kr[i] = make_uint4(0, 0, 0, 0);
            if (at >= 0) {
                if constexpr (SRC == 2) kr[i] = *reinterpret_cast<const uint4 *>(ksrc.row_in_page(pg, at) + (n & (kPieces - 1)) * 8);
                else kr[i] = *reinterpret_cast<const uint4 *>(ksrc.row(at, (n & (kPieces - 1)) == 0) + (n & (kPieces - 1)) * 8);
            }
        }
    };
    auto load_turns = [&](int tile) {
        int pos[4];
        four(sh_pos, tile, pos);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t at = (int64_t)key_id(s0 + tile * 16 + u * 4 + kq, pos[u]) * (kD / 2) + n * 4;
            tc[u] = *reinterpret_cast<const float4 *>(a.rope_cos + at);
            ts[u] = *reinterpret_cast<const float4 *>(a.rope_sin + at);
        }
    };
    auto load_v = [&](int tile) {
        int pos[4], page[4] = {0, 0, 0, 0};
        four(sh_pos, tile, pos);
        if constexpr (SRC == 2) four(sh_page, tile, page);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            vr[u] = v_t{};
            if (pos[u] >= 0) {
                if constexpr (SRC == 2) vr[u] = *reinterpret_cast<const v_t *>(vsrc.row_in_page(page[u], pos[u]) + n * (KV8 ? 4 : 8));
                else vr[u] = *reinterpret_cast<const v_t *>(vsrc.row(pos[u], false) + n * (KV8 ? 4 : 8));      // K did the bookkeeping
            }
        }
    };
    const int tiles = a.slots_per_split >> 4;
    float4 q_cos, q_sin;
    if constexpr (ROPE) {
        block_tokens = sh_block_tokens;
        const int64_t at = (int64_t)max(n_sink_eff + block_tokens + max(0, pr.E - w0) - 1, 0) * (kD / 2) + n * 4;       // (an empty sequence attends to nothing)
        q_cos = *reinterpret_cast<const float4 *>(a.rope_cos + at);
        q_sin = *reinterpret_cast<const float4 *>(a.rope_sin + at);
    }
    if (wv < tiles) {
        load_k(wv);
        if constexpr (ROPE) load_turns(wv);
        load_v(wv);
    }
    float qr[ROPE ? G : 1][8];
    if constexpr (ROPE) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
            unpack8(q_raw[h], qr[h]);
            turn8(qr[h], q_cos, q_sin);
        }
    }
#pragma unroll 1
    for (int tile = wv; tile < tiles; tile += NW) {
        const bool more = tile + NW < tiles;
        f32x4 c[kSets];                       // of column n's head against tokens 4 * kq .. + 3
        if constexpr (ROPE) {
            float d[4][G];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float x[8];
                unpack8(kv[u], x);
                turn8(x, tc[u], ts[u]);
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    d[u][h] = x[0] * qr[h][0];
#pragma unroll
                    for (int i = 1; i < 8; ++i) d[u][h] = fmaf(x[i], qr[h][i], d[u][h]);
                }
            }
            if (more) load_k(tile + NW);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (G <= 4) c[0][u] = head_sum<G>(d[u], n);
                else {
#pragma unroll
                    for (int s = 0; s < kSets; ++s) {
                        const float of[4] = {d[u][4 * s], d[u][4 * s + 1], d[u][4 * s + 2], d[u][4 * s + 3]};
                        c[s][u] = head_sum<4>(of, n);
                    }
                }
            }
        } else {
            // K to operand layout: piece c of row r at c ^ r
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int r = 4 * kq + (KV8 ? 2 * i + (n >> 3) : i);
                stage[r * kPieces + ((n ^ r) & (kPieces - 1))] = kr[i];
            }
            asm volatile("" ::: "memory");        // lanes read what other lanes of the wave wrote (LDS keeps the order)
            if (more) load_k(tile + NW);
            uint4 raw[kLoads];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) raw[i] = stage[n * kPieces + (((i * 4 + kq) ^ n) & (kPieces - 1))];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < kSets; ++s) c[s] = decode_products<KV8, 1>(raw, q[s]);
        }
        int pos[4];
        four(sh_pos, tile, pos);
        const bool ok[4] = {pos[0] >= 0, pos[1] >= 0, pos[2] >= 0, pos[3] >= 0};
        bf16x4 part[kSets][3];                // the four tokens' probabilities, in three parts (24 bits)
#pragma unroll
        for (int s = 0; s < kSets; ++s) {
            float sc[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sc[i] = ok[i] ? c[s][i] * a.scale_log2e : kNegBig;
            const float top = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
            if (__ballot(top > m[s]) != 0) {                    // the reference follows where the scores outgrow it
                const float mn = top > m[s] ? top + kSlack : m[s];
                const float corr = __builtin_amdgcn_exp2f(m[s] - mn);
                m[s] = mn;
                l[s] *= corr;
                const f32x4 ch = {dpp_f32<0x00>(corr), dpp_f32<0x55>(corr), dpp_f32<0xAA>(corr), dpp_f32<0xFF>(corr)};
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int h = 0; h < 4; ++h) acc[s][i][h] *= ch[h];
            }
            float w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = ok[i] ? __builtin_amdgcn_exp2f(sc[i] - m[s]) : 0.f;
            l[s] += (w[0] + w[1]) + (w[2] + w[3]);
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t lo = pack_bf16x2(w[0], w[1]), hi = pack_bf16x2(w[2], w[3]);
                part[s][j] = __builtin_bit_cast(bf16x4, make_uint2(lo, hi));
                if (j == 2) break;
                w[0] -= __uint_as_float(lo << 16); w[1] -= __uint_as_float(lo & 0xffff0000u);       // exact
                w[2] -= __uint_as_float(hi << 16); w[3] -= __uint_as_float(hi & 0xffff0000u);
            }
        }
        uint32_t v[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint4 x = as_bf16x8(vr[u]);
            v[u][0] = x.x; v[u][1] = x.y; v[u][2] = x.z; v[u][3] = x.w;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int w = i >> 1;
            const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
            const bf16x4 vt = __builtin_bit_cast(bf16x4, make_uint2(__builtin_amdgcn_perm(v[1][w], v[0][w], sel), __builtin_amdgcn_perm(v[3][w], v[2][w], sel)));
#pragma unroll
            for (int s = 0; s < kSets; ++s)
#pragma unroll
                for (int j = 2; j >= 0; --j)
                    acc[s][i] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(part[s][j], vt, acc[s][i], 0, 0, 0);
        }
        if (more) {
            if constexpr (ROPE) load_turns(tile + NW);
            load_v(tile + NW);
        }
    }

    // merge the 4 groups of each wave in registers (lanes l, l^16, l^32, l^48 hold the same dims): a
    // row swap hands every lane its own and its partner's value (which of the two is which differs
    // between the partners; the merge is symmetric in them, so both compute the same bits)
    auto both = [](float x, int d, float &a, float &b) {
        const unsigned u = __float_as_uint(x);
        if (d == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
            a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
            a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
        }
    };
    __shared__ float sh_m[NW][G], sh_l[NW][G];
    __shared__ float sh_acc[NW][G][kD];
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
#pragma unroll
        for (int d = 16; d <= 32; d <<= 1) {
            float ma, mb, la, lb;
            both(m[s], d, ma, mb);
            both(l[s], d, la, lb);
            const float mn = fmaxf(ma, mb);
            const float wa = __builtin_amdgcn_exp2f(ma - mn), wb = __builtin_amdgcn_exp2f(mb - mn);
            l[s] = la * wa + lb * wb;
            m[s] = mn;
            const float wah[4] = {dpp_f32<0x00>(wa), dpp_f32<0x55>(wa), dpp_f32<0xAA>(wa), dpp_f32<0xFF>(wa)};
            const float wbh[4] = {dpp_f32<0x00>(wb), dpp_f32<0x55>(wb), dpp_f32<0xAA>(wb), dpp_f32<0xFF>(wb)};
#pragma unroll
            for (int h = 0; h < (G < 4 ? G : 4); ++h)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float xa, xb;
                    both(acc[s][i][h], d, xa, xb);
                    acc[s][i][h] = xa * wah[h] + xb * wbh[h];
                }
        }
        // then the waves through LDS
        if (lane < (G < 4 ? G : 4)) { sh_m[wv][s * 4 + lane] = m[s]; sh_l[wv][s * 4 + lane] = l[s]; }
        if (lane < 16) {
#pragma unroll
            for (int h = 0; h < (G < 4 ? G : 4); ++h)
#pragma unroll
                for (int i = 0; i < 8; ++i) sh_acc[wv][s * 4 + h][n * 8 + i] = acc[s][i][h];
        }
    }
    __syncthreads();

    for (int idx = threadIdx.x; idx < G * kD; idx += kAttnThreads) {
        const int h = idx / kD, c = idx % kD;
        float M = kNegBig;
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) M = fmaxf(M, sh_m[w2][h]);
        float L = 0.f, A = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) {
            const float w = __builtin_amdgcn_exp2f(sh_m[w2][h] - M);
            L = fmaf(w, sh_l[w2][h], L);
            A = fmaf(w, sh_acc[w2][h][c], A);
        }
        a.part_acc[(pbase + h) * kD + c] = A;
        if (c == 0) {
            a.part_ml[(pbase + h) * 2 + 0] = M;
            a.part_ml[(pbase + h) * 2 + 1] = L;
        }
    }
}

// merge the splits: one workgroup per (problem, head), GROUPS x 128 threads, a thread per dim and group; group i takes splits
// i, i + GROUPS, ...  The partial results of a group's first 16 splits (all of them in the usual shapes) are requested at
// once, before anything is computed, and every thread takes the maximum over its splits itself: one trip to
// memory, where a reduction of the maxima first and the sums after it made two dependent trips.  Up to 16 splits one
// group does (no barrier); more take four, whose sums are merged through LDS: 50 splits 11.9 us with one group, 6.2 with four.
constexpr int kMergeAhead = 16;
template <int GROUPS>
__global__ __launch_bounds__(kD * GROUPS) void attn_decode_merge_kernel(const AttnDecodeArgs a)
{
    const int G = a.ge.G;
    const int p = blockIdx.x / G, h = blockIdx.x % G;
    const int c = threadIdx.x % kD, grp = threadIdx.x / kD;
    const int b = p / a.ge.Hkv, g = p % a.ge.Hkv;            // decode: one problem per (sequence, KV head)
    const int64_t pbase = (int64_t)p * a.n_splits * G;
    const float2 *ml = reinterpret_cast<const float2 *>(a.part_ml);
    float2 mlv[kMergeAhead];
    float av[kMergeAhead];
#pragma unroll
    for (int s = 0; s < kMergeAhead; ++s) {
        const int64_t r = pbase + (int64_t)min(s * GROUPS + grp, a.n_splits - 1) * G + h;      // clamped: ignored beyond the last split
        mlv[s] = ml[r];
        av[s] = a.part_acc[r * kD + c];
    }
    float M = kNegBig;
#pragma unroll
    for (int s = 0; s < kMergeAhead; ++s)
        if (s * GROUPS + grp < a.n_splits) M = fmaxf(M, mlv[s].x);
    for (int s = kMergeAhead * GROUPS + grp; s < a.n_splits; s += GROUPS) M = fmaxf(M, ml[pbase + (int64_t)s * G + h].x);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int s = 0; s < kMergeAhead; ++s) {
        if (s * GROUPS + grp < a.n_splits) {
            const float w = __builtin_amdgcn_exp2f(mlv[s].x - M);
            L = fmaf(w, mlv[s].y, L);
            A = fmaf(w, av[s], A);
        }
    }
#pragma unroll 8
    for (int s = kMergeAhead * GROUPS + grp; s < a.n_splits; s += GROUPS) {
        const int64_t r = pbase + (int64_t)s * G + h;
        const float2 x = ml[r];
        const float w = __builtin_amdgcn_exp2f(x.x - M);
        L = fmaf(w, x.y, L);
        A = fmaf(w, a.part_acc[r * kD + c], A);
    }
    if constexpr (GROUPS > 1) {
        __shared__ float sh_m[GROUPS], sh_l[GROUPS], sh_a[GROUPS][kD];
        sh_a[grp][c] = A;
        if (c == 0) { sh_m[grp] = M; sh_l[grp] = L; }
        __syncthreads();
        if (grp != 0) return;
        M = kNegBig;
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) M = fmaxf(M, sh_m[i]);
        L = A = 0.f;
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) {
            const float w = __builtin_amdgcn_exp2f(sh_m[i] - M);
            L = fmaf(w, sh_l[i], L);
            A = fmaf(w, sh_a[i][c], A);
        }
    }
    const int hq = g * G + h;
    a.out[((int64_t)b * a.ge.Hq + hq) * kD + c] = (uint16_t)f32_to_bf16_bits(A / L * a.v_scale);
    if (a.out_lse != nullptr && c == 0)
        a.out_lse[(int64_t)b * a.ge.Hq + hq] = (M + log2f(L)) * 0.69314718055994530942f;
}

// Splits of the slot list: as many workgroups as the chip holds at once, so that no workgroup has to wait for a free place and
// run its whole latency chain after the others have drained -- with 256-slot splits the cfg3 shape
// had 1344 workgroups for 1024 places.  At least 256 slots per split, a multiple of 16; lists that fill the chip several times over go
// in the rounds that take the least time, each as full as can be, and up to 1,536 slots a split are better than a second round that
// is half empty.  At most 1,024 slots a split / so (us): 32 sequences of 5,248 slots, one head a group, E4M3 75.7 / 66.5, four heads, E4M3
// 79.2 / 69.4; 32 of 3,200, four heads, bf16 with RoPE 106.5 / 91.5; 4 of 33,920, one head, E4M3 68.6 / 56.2, bf16 with RoPE 130 / 118.
// (With 64 slots for a split's beginning and end two full rounds win over one that is nearly full, and should not: eight heads, bf16,
// 138 problems of 2,324 slots 43.4 / 38.7.  800 drawn lists: 64, 128 and 256 on the average within 0.3 % of each other.)
// `fine`: where splits of 256 slots would not even give every CU one workgroup, the kernel is one chain of latencies and a
// split walks its loop four times while most of the chip is idle; splits then go down to 64 slots, one batch of loads of
// every 16-lane group, to two workgroups per CU at most (more of them share what a CU has and cost the merge) and to 64 splits,
// which the merge takes in one trip.  Split and merge, 256-slot splits / four workgroups per CU / two (us):
// 4 heads, 8 problems of 1,664 slots 19.4/14.7/15.1, 8 of 5,248 20.7/19.0/19.5, 32 of 1,664 21.0/22.0/19.7; 8 heads
// 25.6/17.8/17.4, 26.7/25.0/24.8, 27.0/30.8/25.1, 16 of 3,200 27.2/30.3/25.4.  Finer splits take more scratch; with
// scratch for the coarse ones only, those are used.
// wg_per_cu: what the instantiation's registers leave room for (attn_decode_per_cu); 0: the most splits of any, which the workspace is
// sized for.
static int decode_splits(const ihip_shape &s, int n_blocks, int block, bool fine, int *slots_per_split, int wg_per_cu)
{
    const int n_cu = compute_units();
    const int total = s.n_sink + n_blocks * block + s.n_stream;
    const int P = std::max(1, s.B * s.Hkv);
    const bool spread = fine && (int64_t)P * ((total + kAttnMinSplit - 1) / kAttnMinSplit) < n_cu;
    auto slots = [&](int splits) { return ((total + splits - 1) / splits + 15) / 16 * 16; };
    if (spread) {
        const int least = std::min(kAttnMinSplit, std::max(kAttnMinSplitFine, ((total + 63) / 64 + 15) & ~15));
        *slots_per_split = std::max(least, slots(std::max(1, n_cu * 2 / P)));
        return (total + *slots_per_split - 1) / *slots_per_split;
    }
    int per = std::min(kAttnUsualSplit, std::max(kAttnMinSplit, slots(std::max(1, n_cu * 4 / P))));
    const int most = (total + per - 1) / per, fewest = (total + kAttnMaxSplit - 1) / kAttnMaxSplit;
    if (wg_per_cu == 0) return most;
    const int64_t places = (int64_t)n_cu * wg_per_cu;
    int64_t best = INT64_MAX;
    for (int64_t rounds = (P * (int64_t)fewest + places - 1) / places, last = rounds + 2; rounds <= last; ++rounds) {
        const int n = slots((int)std::min<int64_t>(most, rounds * places / P)), size = std::max(n, kAttnMinSplit);
        const int64_t time = rounds * (size + kAttnSplitCost);
        if (time < best) {
            best = time;
            per = size;
        }
    }
    *slots_per_split = per;
    return (total + per - 1) / per;
}

// Workgroups on a compute unit: waves per SIMD that the instantiation is compiled for (its launch bounds; eight heads over E4M3 rows fit
// one more).  Eight heads, 16 sequences of 3,200 slots, splits for
// four / for this many: bf16 45.1 / 41.0 us, E4M3 34.5 / 31.0, bf16 with RoPE 60.1 / 52.4.
// E4M3 rows with RoPE and one or two heads: four where the list fills them with splits of the least size, or three larger ones are better.
// One head, 13 problems of 17,536 slots for three / for four (us): 27.4 / 34.4, 26 of them 45.9 / 42.1.
static int attn_decode_per_cu(int G, bool rope, bool fp8, int64_t slots)
{
    if (G == 8) return fp8 && !rope ? 3 : 2;
    const bool four = fp8 && G <= 2 && slots >= (int64_t)4 * kAttnMinSplit * compute_units();
    return rope && !four ? 3 : 4;
}

// scratch for the partial results of the fine or the coarse splits
size_t attn_decode_workspace(const ihip_shape &s, int n_blocks, int block, bool fine)
{
    int per;
    const int ns = decode_splits(s, n_blocks, block, fine, &per, 0);
    const size_t P = (size_t)s.B * s.Hkv;
    const size_t G = s.Hq / s.Hkv;
    return P * ns * G * (2 + kD) * sizeof(float);
}

int32_t launch_attn_decode(const ihip_shape &s, const ihip_tensor &q, const ihip_tensor &k,
                           const ihip_tensor &v, const int32_t *block_starts, int n_blocks, int block,
                           float sm_scale, void *out, float *out_lse, void *ws, bool fine, const BankView *bank,
                           const ihip_rope *rope, hipStream_t st, const KvFormat *fmt)
{
    AttnDecodeArgs a;
    const bool fp8 = fmt && fmt->fp8;
    a.v_scale = fp8 ? fmt->v_scale : 1.0f;
    a.paged = (fmt && fmt->paged.block_table) ? fmt->paged : PagedView{nullptr, 0, 0};
    const bool paged = a.paged.block_table != nullptr;
    if (paged && bank)
        return fail(IHIP_ERR_UNSUPPORTED, "sparse_attn_decode: paged K/V and the host tier exclude each other");
    const bool use_rope = rope && rope->attn_style != IHIP_ROPE_NONE;
    a.rope_cos = a.rope_sin = nullptr;
    if (use_rope) {
        if (rope->attn_style != IHIP_ROPE_STREAMING)
            return fail(IHIP_ERR_INVALID_ARG, "sparse_attn_decode: rope attn_style = %d", rope->attn_style);
        if (!rope->cos || !rope->sin) return fail(IHIP_ERR_INVALID_ARG, "sparse_attn_decode: rope tables are NULL");
        const int64_t need = (int64_t)s.n_sink + (int64_t)n_blocks * block + s.n_stream;   // most keys a query can attend
        if (rope->n_pos < need)
            return fail(IHIP_ERR_INVALID_ARG, "sparse_attn_decode: rope table has %d positions, %lld needed",
                        rope->n_pos, (long long)need);
        a.rope_cos = rope->cos;
        a.rope_sin = rope->sin;
    }
    if (bank && (bank->row_units == kD) == fp8)
        return fail(IHIP_ERR_INVALID_ARG, "sparse_attn_decode: the host tier holds %s rows", fp8 ? "bf16" : "E4M3");
    a.bank = bank ? *bank : BankView{};
    a.ge = make_geometry(s);
    a.q = (const uint16_t *)q.ptr; a.q_sb = q.stride_b; a.q_sh = q.stride_h; a.q_st = q.stride_t;
    a.k = (const uint16_t *)k.ptr; a.k_sb = k.stride_b; a.k_sh = k.stride_h; a.k_st = k.stride_t;
    a.v = (const uint16_t *)v.ptr; a.v_sb = v.stride_b; a.v_sh = v.stride_h; a.v_st = v.stride_t;
    if (fp8) {
        a.k_sb /= 2; a.k_sh /= 2; a.k_st /= 2;      // byte strides (even) in 2-byte units
        a.v_sb /= 2; a.v_sh /= 2; a.v_st /= 2;
    }
    a.block_starts = block_starts;
    a.n_blocks = n_blocks;
    a.block = block;
    a.block_log2 = __builtin_ctz(block);
    a.scale_log2e = sm_scale * 1.44269504088896340736f * (fp8 ? fmt->k_scale : 1.0f);
    const int P = s.B * s.Hkv;
    const int64_t slots = (int64_t)P * (s.n_sink + n_blocks * block + s.n_stream);
    a.n_splits = decode_splits(s, n_blocks, block, fine, &a.slots_per_split, attn_decode_per_cu(a.ge.G, use_rope, fp8, slots));
    const int G = a.ge.G;
    a.part_ml = (float *)ws;
    a.part_acc = a.part_ml + (size_t)P * a.n_splits * G * 2;
    a.out = (uint16_t *)out;
    a.out_lse = out_lse;
    if (P == 0) return IHIP_OK;
    a.grid = decode_grid(a.ge, a.n_splits, bank != nullptr);
    // With RoPE the table is read once for every problem, a row a token, as many bytes as a bf16 K and V.  With the part as the fastest
    // index and a multiple of eight parts an XCD reads an eighth of the table for all problems; otherwise every XCD reads all of it, and it is
    // better that the problems that read the same rows run next to each other, unless they are few (up to 16: 0.89-0.95 of the rate).
    // 26 problems of 17,536 slots, 29 parts, part / problem fastest (us): one head, bf16 67.8 / 56.3, four heads, bf16 69.6 / 58.8, E4M3
    // 49.5 / 45.2; 24 problems, 32 parts 50.4 / 53.0.
    if (use_rope && !bank && P > 16 && a.n_splits % 8 != 0) a.grid.problems_first = a.n_splits <= 65535;
    const dim3 grid = a.grid.dims(P, a.n_splits);
    {
    KernelTimer timer("attn_decode_split", st);
    switch (G) {
#define IHIP_AD_KERNEL(GG, SRCV, RV, F8V)                                                                           \
    hipLaunchKernelGGL((attn_decode_split_kernel<GG, SRCV, RV, F8V>), grid, dim3(kAttnThreads), 0, st, a)
#define IHIP_AD_BY_FMT(GG, SRCV)                                                                                    \
    if (use_rope && fp8) IHIP_AD_KERNEL(GG, SRCV, true, true);                                                      \
    else if (use_rope) IHIP_AD_KERNEL(GG, SRCV, true, false);                                                       \
    else if (fp8) IHIP_AD_KERNEL(GG, SRCV, false, true);                                                            \
    else IHIP_AD_KERNEL(GG, SRCV, false, false)
#define IHIP_AD_LAUNCH(GG)                                                                                          \
    if (bank) { IHIP_AD_BY_FMT(GG, 1); }                                                                            \
    else if (paged) { IHIP_AD_BY_FMT(GG, 2); }                                                                      \
    else { IHIP_AD_BY_FMT(GG, 0); }
    case 1: IHIP_AD_LAUNCH(1); break;
    case 2: IHIP_AD_LAUNCH(2); break;
    case 4: IHIP_AD_LAUNCH(4); break;
    case 8: IHIP_AD_LAUNCH(8); break;
#undef IHIP_AD_LAUNCH
#undef IHIP_AD_BY_FMT
#undef IHIP_AD_KERNEL
    default: return fail(IHIP_ERR_UNSUPPORTED, "Hq/Hkv = %d not in {1,2,4,8}", G);
    }
    }
    int32_t rc = check_launch("sparse_attn_decode (split)");
    if (rc != IHIP_OK) return rc;
    KernelTimer timer("attn_decode_merge", st);
    if (a.n_splits <= kMergeAhead) hipLaunchKernelGGL(attn_decode_merge_kernel<1>, dim3(P * G), dim3(kD), 0, st, a);
    else hipLaunchKernelGGL(attn_decode_merge_kernel<4>, dim3(P * G), dim3(kD * 4), 0, st, a);
    return check_launch("sparse_attn_decode (merge)");
}

}  // namespace ihip
