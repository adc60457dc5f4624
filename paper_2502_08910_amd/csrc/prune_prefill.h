// Pruning-stage scoring for chunked prefill (Alg. 2 / Alg. 3 with b_q = 16, 32 or 64 queries per
// block): the kernel template and its launcher, shared by the bf16 and the E4M3 translation units.
#pragma once

#include "prune_args.h"
#include <type_traits>

namespace ihip {

// ---------------------------------------------------------------------------
// Chunked-prefill kernel (b_q = 16*MT queries per block).  The score of a key
// is max_t q_t . k over the block's queries: a [b_q x 128] x [128 x 16] matrix
// product per 16 candidate keys, done on the matrix cores
// (v_mfma_f32_16x16x32_bf16; queries are the rows, candidates the columns, so
// the max over queries is an in-lane max over the accumulator plus two
// cross-lane steps).  One wave per query head, G waves per workgroup; a wave
// walks the searches of NT*16 chunks at a time, one candidate row per chunk
// and level.  Workgroups are ordered so that all query blocks and KV heads
// sweep the same chunk range together: the K rows they share stay in L2.
// Operand layout: lane l holds 8 consecutive dims (kq = l/16) of row/column
// l%16; accumulator lane l holds column l%16, rows 4*(l/16)..+3.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kPrefillMaxIters = 4;     // chunk groups (of 32 chunks) per workgroup, at most

//
// ROPE: relative-style dynamic RoPE (Sec. 4 "Dynamic RoPE for OOL generalization"; ApplyRopeQ /
// ApplyRopeK after Alg. 3).  Every query of the block sits at n_stream+1, a left-branch key at 0,
// a right-branch key (and the representative in the chunk score) at 1.  With a table of true
// rotations the key rotations fold into the queries: two rotated copies of the query operands,
// q_L = R(n_stream+1) q and q_R = R(n_stream) q (rounded to bf16 for the matrix cores), and every
// candidate row is scored against both, because a key that wins as the right branch is the left
// branch of the next iteration.  Twice the matrix work and twice the query registers: blocks of 16 and
// 32 queries (64-query blocks: prune_relative.h).
//
// Precision of the rotated operands: a rotated vector is kept as two bf16 operands, its rounded
// value and the rounded rest (rotate_bf16x8_split), and the products of the rests with the other
// side's rounded values are added on the matrix cores as well, so that a score agrees with the
// product of the fp32 rotations to about 2^-16 relative and a selection is decided as an fp32
// evaluation decides it.  Relative style: both rotated query sets have a rest (the keys are not
// rotated: exact), twice the matrix work again.  Chunk-indexed style: the keys have one (q.k_hi + q.k_lo),
// twice the plain kernel's matrix work; the rests of a key tile live in a second LDS tile.
//
// ROPE == 2: chunk-indexed style.  Every key of chunk j (index in the stage's chunk list) sits at
// j, query t of the block at min(its own position, cap) with cap = n_chunk - 1 + n_stream.  With a table of true
// rotations only differences of positions matter, so everything is turned back by cap: the keys of
// chunk j by cap - j, a query by cap - its position, which is nothing at all for a block whose first
// query is at or behind the cap -- every block but those of ranges that hold fewer keys than a block has queries.
// Such queries stay the exact bf16 values they are: no second operand for them, a third of the matrix
// work less than with rotated queries, and 64 registers less, which makes room for two and three waves per SIMD.
// (Blocks before the cap turn their query operands where they are used, value and rest.)
// A candidate row is turned on its way from global memory to LDS, each lane the 16 bytes it fetched
// (tile row 4r + kq is candidate column 4(r%4) + kq of tile r/4, whose chunk and therefore table row
// are the same at every level of a search: the 8 table pieces of a lane are fetched once per chunk
// group); the value goes to the tile, the rest to a second tile.  Same carried-score search as the plain kernel.
// What bounds it: the rotations' vector instructions (40 for 8 values: 48 with the rests by shift, mask and subtraction), then the
// matrix work.  4,096 queries on 128K keys, chunks of 64, 32 heads: 2267 us with rotated queries and keys (three products, one
// wave per SIMD, rows turned in LDS), 1312 us this way with 32 rows at a time and the turns in registers, 1180 with 16 (kTurn16).  Error against 64 bits on the same shape, twelve inputs: searches that end in another leaf
// (near ties) 178 -> 95 of 12.7 million scores, all other scores 1.47e-6 -> 8.2e-7 relative.
__device__ inline void rotate_operand_split(const bf16x8 x, const float4 c, const float4 sn, bf16x8 &hi, bf16x8 &lo)
{
    uint4 h, l;
    rotate_bf16x8_split(__builtin_bit_cast(uint4, x), c, sn, h, l);
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}
__device__ inline void rotate_operand_split(const bf16x8 x, const float *cos4, const float *sin4, bf16x8 &hi,
                                            bf16x8 &lo)
{
    rotate_operand_split(x, *reinterpret_cast<const float4 *>(cos4), *reinterpret_cast<const float4 *>(sin4), hi, lo);
}

// The inverse rotation (sin negated), kept to twice the mantissa like rotate_f32x8_split; the sums are fused
// multiply-adds here (the kernel's time is its vector instructions).
__device__ inline void turn_back_f32x8_split(const float (&f)[8], const float4 c, const float4 sn, uint4 &hi, uint4 &lo)
{
    const float cc[4] = {c.x, c.y, c.z, c.w}, ss[4] = {sn.x, sn.y, sn.z, sn.w};
    uint32_t wh[4], wl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float e = f[2 * i], o = f[2 * i + 1];
        const float re = __fmaf_rn(e, cc[i], __fmul_rn(o, ss[i]));
        const float ro = __fmaf_rn(o, cc[i], -__fmul_rn(e, ss[i]));
        wh[i] = pack_bf16x2(re, ro);
        // re - hi and ro - hi, exact, one v_dot2_f32_bf16 each against (-1, 0) and (0, -1).  (The constants come from registers: as
        // an inline constant the first one reaches the instruction in the other half.)
        uint32_t minus_low = 0x0000bf80u, minus_high = 0xbf800000u;
        asm("" : "+s"(minus_low), "+s"(minus_high));
        const bf16x2_t h2 = __builtin_bit_cast(bf16x2_t, wh[i]);
        wl[i] = pack_bf16x2(__builtin_amdgcn_fdot2_f32_bf16(h2, __builtin_bit_cast(bf16x2_t, minus_low), re, false),
                            __builtin_amdgcn_fdot2_f32_bf16(h2, __builtin_bit_cast(bf16x2_t, minus_high), ro, false));
    }
    hi = make_uint4(wh[0], wh[1], wh[2], wh[3]);
    lo = make_uint4(wl[0], wl[1], wl[2], wl[3]);
}
__device__ inline void turn_back_split(const uint4 x, const float4 c, const float4 sn, uint4 &hi, uint4 &lo)
{
    float f[8];
    unpack_bf16x8(x, f);
    turn_back_f32x8_split(f, c, sn, hi, lo);
}
__device__ inline void turn_back_split(const uint2 x, const float4 c, const float4 sn, uint4 &hi, uint4 &lo)
{
    float f[8];
    unpack8_fp8(x, f);
    turn_back_f32x8_split(f, c, sn, hi, lo);
}
__device__ inline void turn_back_operand_split(const bf16x8 x, const float *cos4, const float *sin4, bf16x8 &hi,
                                               bf16x8 &lo)
{
    uint4 h, l;
    turn_back_split(__builtin_bit_cast(uint4, x), *reinterpret_cast<const float4 *>(cos4),
                    *reinterpret_cast<const float4 *>(sin4), h, l);
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

// PAGED: K is a page pool read through the sequence's row of the block table: the lane that owns a
// candidate looks its page up and forms the row's element offset (64-bit) before the offsets are
// handed to the loading lanes, so a level costs one more dependent (cache-resident) load.
//
// KV8: K rows are 128 bytes of E4M3.  There is no 8-byte direct-to-LDS load, so a lane fetches its 8
// bytes of a row into registers, repacks them as bf16 (exact) and stores the 16 bytes where the
// direct load would have put them (chunk-indexed RoPE: rotated on the way, which saves the round
// trip through LDS); everything after that is the bf16 kernel.  The chunk score is multiplied by the
// tensor's scale at the end.  K strides count 2-byte units.
//
// FEW: chunk-indexed RoPE, 64-query blocks, four waves: registers for two waves per SIMD instead of three, without scratch, where
// there are no workgroups for a third
template <int MT, int NT, int G, bool WIDE, int ROPE, bool PAGED, int PARTS = 1, bool KV8 = false, bool FEW = false>
__global__ __launch_bounds__(64 * G, ROPE == 2 ? (G == 4 && PARTS == 1 && !FEW ? 3 : 2) : (ROPE || (KV8 && PARTS > 1)) ? 2 : (PARTS == 1) ? 4 : 3) void prune_prefill_kernel(const PruneArgs a, const int iters,
                                                                            const RopeView rope)
{
    static_assert(NT == 2, "the shared first phase assumes two 16-chunk tiles per wave");
    static_assert(!PAGED || WIDE, "paged pools are addressed with 64-bit offsets");
    static_assert(ROPE != 1 || MT <= 2, "64-query blocks with the relative style have a kernel of their own");
    constexpr int NWV = G;                           // waves of the workgroup
    constexpr int MTW = MT;                          // 16-query tiles of a wave
    constexpr int kTile = NT * 16 * kD;              // one tile: 32 rows of 256 bytes, no padding
    constexpr bool kShare = NWV >= 2;                // two tiles are needed for the shared phase
    __shared__ float sh_sigma[2][G][NT * 16];       // two buffers: a chunk group writes while the last one is still read
    __shared__ float sh_best[kPrefillMaxIters][NT * 16];      // chunk scores over the head parts done so far
    // ROPE == 2, workgroups of four waves: a wave turns and scores 16 rows at a time, values and then rests in its tile (in the shared
    // first phase the rests of the two tiles lie behind them), and the turns of a chunk group are in LDS for all waves, [cos, sin]
    // [chunk][piece].  49 KB and 168 registers: three workgroups on a compute unit, three waves per SIMD (64-query blocks, 100 bytes of scratch per lane;
    // two where the launch has no more, 20.9 / 18.4 us for 16 problems, and for two passes of four heads, 297 / 277).  Other workgroups
    // turn 32 rows at a time, rests in a second tile, each lane's turns in registers, two waves per SIMD: one and two waves
    // share a table too little, eight would not fit three times.  Registers / LDS: four heads, 64-query blocks, chunks of 64, 4,096
    // queries on 128K keys 1302 / 1169 us, 32-query blocks (1,024 on 32K) 66 / 60, 16 99 / 89; two heads 63 / 67, one 64 / 110.
    constexpr bool kTurn16 = ROPE == 2 && NWV == 4;
    constexpr int kLo = kTurn16 ? 16 * kD : ROPE == 2 ? NWV * kTile : 0, kLoShared = kTurn16 ? 2 * kTile : kLo;
    __shared__ __attribute__((aligned(16))) uint16_t sh_rows[(ROPE == 2 && !kTurn16 ? 2 * NWV : NWV) * kTile];
    __shared__ float4 sh_table[kTurn16 ? 2 : 1][kTurn16 ? NT * 16 * 16 : 1];
    float4 tb_cos[ROPE == 2 && !kTurn16 ? NT * 4 : 1], tb_sin[ROPE == 2 && !kTurn16 ? NT * 4 : 1];
    // Workgroups are dealt to the 8 XCDs round-robin by linear id; let the KV head be the fastest
    // index, so that (with 8 KV heads) one XCD's L2 only ever holds one head's K rows and all
    // query blocks that share those rows run on that XCD at about the same time.
    const int p = ((blockIdx.x / a.ge.Hkv / a.ge.Mq) * a.ge.Hkv + blockIdx.x % a.ge.Hkv) * a.ge.Mq +
                  (blockIdx.x / a.ge.Hkv) % a.ge.Mq;
    const Problem pr = problem_of(a.ge, p);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int n = lane & 15, kq = lane >> 4;
    // G is the number of heads (waves) a pass works on; a group of G*PARTS heads (8, where 8 waves
    // of this many registers would leave room for one workgroup per CU only) is done in PARTS
    // passes, one after the other, by the same waves
    constexpr int parts = PARTS;
    int h = pr.g * (G * PARTS) + wv;
    using raw_t = typename std::conditional<KV8, uint2, uint4>::type;         // a lane's 8 elements of a row as fetched
    constexpr bool kViaRegs = KV8 || ROPE == 2;      // rows are worked on between global memory and LDS
    using off_t = typename std::conditional<WIDE, int64_t, uint32_t>::type;   // element offset of a row
    const off_t k_st = (off_t)a.k_st;

    // Rows travel from global memory straight into LDS (global_load_lds, 16 bytes per lane: 16
    // lanes fetch one whole 256-byte row, 4 rows per instruction, landing at base + lane*16) and
    // are re-read from there in the MFMA operand layout (lane = (row or column n, 8 dims of group
    // kq)).  Reading them from global memory in that layout costs four times as many L1 accesses
    // per row and makes the L1 tag rate the bound; staging through registers costs 32 VGPRs and 8
    // LDS stores per phase.  The LDS destination of a lane is fixed, so the bank swizzle is applied
    // on the source side: 16-byte slot c of tile row R holds dims 8*(c ^ (R%16)).., which makes the
    // 16 rows of an operand read hit 16 different bank groups.
    // load4(base, stride, dst, row, swz): lanes 16*kq..+15 fetch row `row` (their own copy of it)
    // to the tile row dst + kq; dst is the LDS byte address of a four-row group, wave-uniform.
    // "No candidate" is row 0 (always readable; the lane that owns the candidate substitutes it) and
    // the caller ignores the score, which keeps the loads free of branches: with exec-masked loads
    // every shuffle result has to be waited for on its own.  The instruction is written as
    // assembly so that the destinations can be computed once, outside the search loops.
    // Narrow offsets: the base is wave-uniform (scalar registers) and the lane's byte offset one
    // 24-bit multiply and an add, the load's scalar-base form.
    // `row` is never negative here: the lane that owns a candidate passes row 0 for "no candidate".
    auto load4 = [&](const uint16_t *base, off_t stride, uint32_t dst, int row, int swz) {
        const off_t r = (off_t)row;
        if constexpr (WIDE) {
            global_to_lds(dst, base + r * stride + ((n ^ swz) << 3));
        } else {
            global_to_lds(dst, base, __umul24((uint32_t)r, (uint32_t)stride * 2u) + (uint32_t)((n ^ swz) << 4));
        }
    };
    // the same with the row's element offset already formed (paged K)
    auto load4_at = [&](const uint16_t *base, int64_t at, uint32_t dst, int swz) {
        global_to_lds(dst, base + at + ((n ^ swz) << 3));
    };
    // Keys that go through registers (E4M3, chunk-indexed RoPE): this lane's 8 elements of row `row` (or of the
    // row at element offset `at`), and their place in a four-row group of a tile
    auto fetch = [&](const uint16_t *base, off_t stride, int row, int swz) {
        const off_t r = (off_t)max(row, 0);
        const off_t at = WIDE ? r * stride : (off_t)__umul24((uint32_t)r, (uint32_t)stride);
        return *reinterpret_cast<const raw_t *>(base + at + (n ^ swz) * (int)(sizeof(raw_t) / 2));
    };
    auto fetch_at = [&](const uint16_t *base, int64_t at, int swz) {
        return *reinterpret_cast<const raw_t *>(base + at + (n ^ swz) * (int)(sizeof(raw_t) / 2));
    };
    auto put16 = [&](uint16_t *four_rows, const uint4 piece) {
        *reinterpret_cast<uint4 *>(four_rows + kq * kD + n * 8) = piece;
    };
    auto lds_addr = [&](const uint16_t *ptr) {
        return (uint32_t)__builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)ptr);
    };
    auto operand = [&](const uint16_t *tile, int row16, int ks) {
        return *reinterpret_cast<const bf16x8 *>(&tile[(row16 + n) * kD + (((ks << 2) + kq) ^ n) * 8]);
    };

    // A operands: the block's queries, [MT tiles of 16 rows] x [4 steps of 32 dims], staged
    // through this wave's own tile, 32 rows at a time
    uint16_t *tile = &sh_rows[wv * kTile];
    uint32_t dst_own[NT * 4];                        // this wave's tile, four rows at a time
#pragma unroll
    for (int r = 0; r < NT * 4; ++r) dst_own[r] = lds_addr(tile + r * 4 * kD);
    bf16x8 qa[MTW][4];                               // relative RoPE: q_L
    bf16x8 qaR[ROPE == 1 ? MTW : 1][4];              // relative RoPE: q_R
    bf16x8 qaLo[ROPE == 1 ? MTW : 1][4];             // relative RoPE: what rounding the rotated queries to bf16 dropped
    bf16x8 qaRLo[ROPE == 1 ? MTW : 1][4];
    int q_cap = 0;                                   // chunk-indexed RoPE: the largest query position
    bool q_capped = true;                            // ... and whether every query of the block sits there
    if constexpr (ROPE == 2) {
        __shared__ int sh_n_chunk;
        q_cap = stage_n_chunk(a, pr, p, 64 * NWV, &sh_n_chunk) - 1 + a.ge.n_stream;
        q_capped = pr.E - a.ge.b_q >= q_cap;
    }
    auto stage_queries = [&]() {
        const uint16_t *qb = a.q + pr.b * a.q_sb + (int64_t)h * a.q_sh + (int64_t)(pr.m * a.ge.b_q) * a.q_st;
        // PARTS > 1: the row addresses are formed here, not carried over the passes.  Carried, they cost the chunk-indexed
        // style up to 512 bytes of scratch per lane: 64-query blocks, 8 heads, pages 902 -> 444 us a layer (1,024 queries
        // on 32K keys; E4M3 pages 847 -> 573, contiguous rows 465 -> 391)
        int row0 = 0;
        if constexpr (PARTS > 1) asm volatile("" : "+v"(row0));
#pragma unroll
        for (int m0 = 0; m0 < MTW; m0 += 2) {
            constexpr int kRows = MTW >= 2 ? 32 : 16;
#pragma unroll
            for (int r = 0; r < kRows / 4; ++r)
                load4(qb, (off_t)a.q_st, dst_own[r], row0 + m0 * 16 + r * 4 + kq, (r & 3) * 4 + kq);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int mt = m0; mt < m0 + 2 && mt < MTW; ++mt)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    qa[mt][ks] = operand(tile, (mt - m0) * 16, ks);
                    if constexpr (ROPE == 1) {
                        const int pair = ((ks << 2) + kq) * 4;       // first of this operand's 4 dim pairs
                        const int64_t posR = (int64_t)a.ge.n_stream * (kD / 2) + pair, posL = posR + kD / 2;
                        rotate_operand_split(qa[mt][ks], rope.cos + posR, rope.sin + posR, qaR[mt][ks], qaRLo[mt][ks]);
                        rotate_operand_split(qa[mt][ks], rope.cos + posL, rope.sin + posL, qa[mt][ks], qaLo[mt][ks]);
                    }
                }
            // the reads must have left LDS before the next loads land in the same tile
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    };
    if constexpr (PARTS == 1) {
        stage_queries();
        if (kShare) __syncthreads();                 // other waves' tiles are written below
    }
    const uint16_t *kb = PAGED ? a.k + pr.g * a.k_sh : a.k + pr.b * a.k_sb + pr.g * a.k_sh;
    const int32_t *table = PAGED ? a.paged.block_table + (int64_t)pr.b * a.paged.table_stride : nullptr;
    const int page_mask = PAGED ? (1 << a.paged.page_log2) - 1 : 0;
    // paged K: element offset of row `pos` from kb (a row of -1 stands for row 0, as in load4)
    auto paged_at = [&](int pos) {
        const int r = max(pos, 0);
        return (int64_t)table[r >> a.paged.page_log2] * a.k_sb + (int64_t)(r & page_mask) * a.k_st;
    };

    // Chunk-indexed RoPE, blocks with queries before the cap: the queries are read again, turned back to the cap (value
    // and rest) and used at once, with nothing kept in registers.
    auto scores_before_cap = [&](const uint16_t *src, int lo_at) {
        const uint16_t *qb = a.q + pr.b * a.q_sb + (int64_t)h * a.q_sh + (int64_t)(pr.m * a.ge.b_q) * a.q_st;
        float best = -INFINITY;
#pragma unroll 1
        for (int mt = 0; mt < MTW; ++mt) {
            const int row = mt * 16 + n;
            const int64_t back = (int64_t)max(q_cap - (pr.E - a.ge.b_q + row), 0) * (kD / 2);
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int ks = 0; ks < 4; ++ks) {
                const int piece = (ks << 2) + kq;
                const bf16x8 q = *reinterpret_cast<const bf16x8 *>(qb + (int64_t)row * a.q_st + piece * 8);
                bf16x8 hi, lo;
                turn_back_operand_split(q, rope.cos + back + piece * 4, rope.sin + back + piece * 4, hi, lo);
                const bf16x8 k = operand(src, 0, ks), k_rest = operand(src + lo_at, 0, ks);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, k, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, k_rest, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, k, c, 0, 0, 0);
            }
            best = fmaxf(best, fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
        }
        return max_over_rows(best);
    };
    // chunk-indexed RoPE: scores of 16 turned rows (values at src, rests lo_at behind them)
    auto turned_scores = [&](const uint16_t *src, int lo_at) {
        if (!q_capped) return scores_before_cap(src, lo_at);
        bf16x8 kr[4], kr_rest[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            kr[ks] = operand(src, 0, ks);
            kr_rest[ks] = operand(src + lo_at, 0, ks);
        }
        float best = -INFINITY;
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};          // the small terms first
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[mt][ks], kr_rest[ks], c, 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[mt][ks], kr[ks], c, 0, 0, 0);
            best = fmaxf(best, fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
        }
        return max_over_rows(best);
    };
    // scores of the 32 rows of a tile (column n of 16-row tile t): max over the block's queries
    // (ROPE: sig against q_L, sigR against q_R)
    auto mfma_scores = [&](const uint16_t *src, float (&sig)[NT], float (&sigR)[NT]) {      // (kTurn16: of the shared first phase)
        if constexpr (ROPE == 2) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                sig[t] = turned_scores(src + t * 16 * kD, kLoShared);
                if constexpr (MT > 1 || kTurn16) __builtin_amdgcn_sched_barrier(0);      // one tile's operands at a time
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            bf16x8 kr[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kr[ks] = operand(src, t * 16, ks);
            float best = -INFINITY, bestR = -INFINITY;
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt) {
                f32x4 c = {0.f, 0.f, 0.f, 0.f};
                if constexpr (ROPE == 1) {           // the small terms first
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qaLo[mt][ks], kr[ks], c, 0, 0, 0);
                }
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[mt][ks], kr[ks], c, 0, 0, 0);
                best = fmaxf(best, fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
                if constexpr (ROPE == 1) {
                    f32x4 cr = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        cr = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qaRLo[mt][ks], kr[ks], cr, 0, 0, 0);
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        cr = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qaR[mt][ks], kr[ks], cr, 0, 0, 0);
                    bestR = fmaxf(bestR, fmaxf(fmaxf(cr[0], cr[1]), fmaxf(cr[2], cr[3])));
                }
            }
            sig[t] = max_over_rows(best);
            if constexpr (ROPE == 1) {
                sigR[t] = max_over_rows(bestR);
            }
        }
    };
    // table piece of this lane for load instruction r of the chunk group at jt: chunk j's keys are
    // turned back by q_cap - j
    auto table_at = [&](int jt, int r) {
        const int j = jt + (r >> 2) * 16 + (r & 3) * 4 + kq;
        return (int64_t)max(q_cap - j, 0) * (kD / 2) + ((n ^ ((r & 3) * 4 + kq)) << 2);
    };
    // score of candidate rows pos[t] of this wave's own searches.  The scores of columns whose
    // search has ended are ignored by the caller.
    auto score = [&](const int (&pos)[NT], const bool (&ok)[NT], float (&sig)[NT], float (&sigR)[NT]) {
        if constexpr (kViaRegs) {
            raw_t raw[NT * 4];
            if constexpr (PAGED) {
                int64_t at[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) at[t] = paged_at(ok[t] ? pos[t] : -1);
#pragma unroll
                for (int r = 0; r < NT * 4; ++r)
                    raw[r] = fetch_at(kb, __shfl(at[r >> 2], (r & 3) * 4 + kq, 64), (r & 3) * 4 + kq);
            } else {
#pragma unroll
                for (int r = 0; r < NT * 4; ++r)
                    raw[r] = fetch(kb, k_st, __shfl(ok[r >> 2] ? pos[r >> 2] : -1, (r & 3) * 4 + kq, 64),
                                   (r & 3) * 4 + kq);
            }
            if constexpr (kTurn16) {
                // 16 rows at a time: turned (one piece after the other: registers), stored, scored
#pragma unroll
                for (int t = 0; t < NT; ++t) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int at = (t * 16 + i * 4 + kq) * 16 + (n ^ (i * 4 + kq));
                        uint4 piece, rest;
                        turn_back_split(raw[t * 4 + i], sh_table[0][at], sh_table[1][at], piece, rest);
                        put16(tile + i * 4 * kD, piece);
                        put16(tile + kLo + i * 4 * kD, rest);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // the wave reads back what its other lanes stored: LDS serves a wave's requests in order
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    sig[t] = turned_scores(tile, kLo);
                    asm volatile("" ::: "memory");
                }
                return;
            }
#pragma unroll
            for (int r = 0; r < NT * 4; ++r) {
                uint4 piece;
                if constexpr (ROPE == 2) {
                    uint4 rest;
                    turn_back_split(raw[r], tb_cos[kTurn16 ? 0 : r], tb_sin[kTurn16 ? 0 : r], piece, rest);
                    put16(tile + kLo + r * 4 * kD, rest);
                } else {
                    piece = as_bf16x8(raw[r]);
                }
                put16(tile + r * 4 * kD, piece);
                if constexpr (ROPE == 2) __builtin_amdgcn_sched_barrier(0);      // one piece after the other: registers
            }
            // the wave reads back what its other lanes stored: LDS serves a wave's requests in order
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            mfma_scores(tile, sig, sigR);
            return;
        }
        if constexpr (PAGED) {
            int64_t at[NT], cand_at[NT * 4];
#pragma unroll
            for (int t = 0; t < NT; ++t) at[t] = paged_at(ok[t] ? pos[t] : -1);
#pragma unroll
            for (int r = 0; r < NT * 4; ++r) cand_at[r] = __shfl(at[r >> 2], (r & 3) * 4 + kq, 64);
#pragma unroll
            for (int r = 0; r < NT * 4; ++r) load4_at(kb, cand_at[r], dst_own[r], (r & 3) * 4 + kq);
        } else {
            int cand[NT * 4];
#pragma unroll
            for (int r = 0; r < NT * 4; ++r)     // lanes 0..15 hold column = lane
                cand[r] = __shfl(ok[r >> 2] ? pos[r >> 2] : 0, (r & 3) * 4 + kq, 64);
#pragma unroll
            for (int r = 0; r < NT * 4; ++r)     // tile row r*4 + kq = candidate (t = r/4, column (r%4)*4 + kq)
                load4(kb, k_st, dst_own[r], cand[r], (r & 3) * 4 + kq);
        }
        // the loads count on vmcnt; the wave reads its own tile, so no barrier is needed
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        mfma_scores(tile, sig, sigR);
    };

    // destinations of this wave's share of the loads of the shared first phase
    uint32_t dst_shared[kShare ? 16 / NWV : 1];
#pragma unroll
    for (int i = 0; i < (kShare ? 16 / NWV : 1); ++i) dst_shared[i] = lds_addr(&sh_rows[(wv * (16 / NWV) + i) % (NWV * 8) * 4 * kD]);
    for (int part = 0; part < parts; ++part) {
    if constexpr (PARTS > 1) {
        h = pr.g * (G * PARTS) + part * G + wv;
        stage_queries();
        if (kShare) __syncthreads();                 // other waves' tiles are written below
    }
    for (int it = 0; it < iters; ++it) {
        const int jt = (blockIdx.y * iters + it) * NT * 16;
        int start[NT], len[NT], off[NT], pos[NT];
        bool valid[NT], ok[NT];
        float sigma[NT], s[NT];                      // chunk score so far; scores of the candidates
        float sL[NT], sR[NT];                        // ROPE: the current left key against q_L; candidates against q_R
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int j = jt + t * 16 + n;
            start[t] = j < a.max_chunks
                           ? slot_start(pr, a.parent_starts, a.n_parent, a.ratio_log2, a.chunk, p, j)
                           : -1;
            valid[t] = start[t] >= 0;
            len[t] = valid[t] ? min(a.chunk, pr.hi - start[t]) : 0;
            off[t] = 0;
            pos[t] = start[t];
        }
        auto load_table = [&]() {
            if constexpr (ROPE == 2 && !kTurn16) {
#pragma unroll
                for (int r = 0; r < NT * 4; ++r) {
                    const int64_t at = table_at(jt, r);
                    tb_cos[kTurn16 ? 0 : r] = *reinterpret_cast<const float4 *>(rope.cos + at);
                    tb_sin[kTurn16 ? 0 : r] = *reinterpret_cast<const float4 *>(rope.sin + at);
                }
            }
        };
        // 16-query blocks multiply too little to cover the table's way from memory, and have the registers for it: asked
        // for ahead of the first keys (that and both tiles' operands at once above: two heads per group 164 -> 149 us)
        constexpr bool kTableFirst = MT == 1;
        if constexpr (kTableFirst) load_table();
        // kTurn16: the chunk group's turns are requested ahead of the first keys and stored once those are on their way
        // (every wave has left the last group's: the barrier at its end)
        constexpr int kTurns = kTurn16 ? NT * 16 * 16 / (64 * NWV) : 1;
        float4 turn_cos[kTurns], turn_sin[kTurns];
        if constexpr (kTurn16) {
#pragma unroll
            for (int i = 0; i < kTurns; ++i) {
                const int item = (int)threadIdx.x + i * 64 * NWV;
                const int64_t at = (int64_t)max(q_cap - (jt + (item >> 4)), 0) * (kD / 2) + ((item & 15) << 2);
                turn_cos[i] = *reinterpret_cast<const float4 *>(rope.cos + at);
                turn_sin[i] = *reinterpret_cast<const float4 *>(rope.sin + at);
            }
        }
        int half = a.chunk >> 1;
        if (kShare) {
            // The first key of a chunk and of its right half are the same rows for every head of
            // the group: the waves fetch them together, once (tile 0: first keys, tile 1: first
            // keys of the right halves; 16 four-row loads dealt evenly to the G waves), and each
            // wave scores both tiles against its own queries.
            constexpr int kPerWave = 16 / NWV;
            int cand[kPerWave];
            int64_t cand_at[PAGED ? kPerWave : 1];
#pragma unroll
            for (int i = 0; i < kPerWave; ++i) {
                const int ld = wv * kPerWave + i;                    // wave-uniform
                const int set = ld >> 3, r = ld & 7;
                const int st_ = (r >> 2) ? start[1] : start[0], ln_ = (r >> 2) ? len[1] : len[0];
                const int c = set == 0 ? st_ : (half >= 1 && half < ln_ ? st_ + half : -1);
                if constexpr (PAGED) cand_at[i] = __shfl(paged_at(c), (r & 3) * 4 + kq, 64);
                else cand[i] = __shfl(max(c, 0), (r & 3) * 4 + kq, 64);
            }
            if constexpr (kViaRegs) {
                raw_t raw[kPerWave];
#pragma unroll
                for (int i = 0; i < kPerWave; ++i) {
                    const int r = (wv * kPerWave + i) & 7;
                    if constexpr (PAGED) raw[i] = fetch_at(kb, cand_at[i], (r & 3) * 4 + kq);
                    else raw[i] = fetch(kb, k_st, cand[i], (r & 3) * 4 + kq);
                }
                if constexpr (kTurn16) {
#pragma unroll
                    for (int i = 0; i < kTurns; ++i) {
                        sh_table[0][(int)threadIdx.x + i * 64 * NWV] = turn_cos[i];
                        sh_table[1][(int)threadIdx.x + i * 64 * NWV] = turn_sin[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < kPerWave; ++i) {
                    const int ld = wv * kPerWave + i;
                    uint4 piece;
                    if constexpr (ROPE == 2) {
                        const int64_t at = table_at(jt, ld & 7);
                        uint4 rest;
                        turn_back_split(raw[i], *reinterpret_cast<const float4 *>(rope.cos + at),
                                        *reinterpret_cast<const float4 *>(rope.sin + at), piece, rest);
                        put16(&sh_rows[kLoShared + ld * 4 * kD], rest);
                    } else {
                        piece = as_bf16x8(raw[i]);
                    }
                    put16(&sh_rows[ld * 4 * kD], piece);
                    if constexpr (ROPE == 2) __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
            for (int i = 0; i < kPerWave; ++i) {
                const int r = (wv * kPerWave + i) & 7;
                if constexpr (PAGED) load4_at(kb, cand_at[i], dst_shared[i], (r & 3) * 4 + kq);
                else load4(kb, k_st, dst_shared[i], cand[i], (r & 3) * 4 + kq);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            __syncthreads();
            if constexpr (!kTableFirst) load_table();        // for the waves' own searches; there when the tiles below are scored
            float l0r[NT];
            mfma_scores(&sh_rows[0], sigma, l0r);
            mfma_scores(&sh_rows[kTile], s, sR);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bool has_right = half >= 1 && half < len[t];
                if constexpr (ROPE == 1) {
                    const bool right = has_right && sR[t] > sigma[t];        // strict: tie keeps left
                    off[t] = right ? half : 0;
                    sL[t] = right ? s[t] : sigma[t];
                    sigma[t] = right ? sR[t] : l0r[t];
                } else if (has_right && s[t] > sigma[t]) { off[t] = half; sigma[t] = s[t]; }
            }
            half >>= 1;
            __syncthreads();                         // tiles 0 and 1 go back to their waves
        } else {
            if constexpr (!kTableFirst) load_table();
            score(pos, valid, sigma, sR);
            if constexpr (ROPE == 1) {
#pragma unroll
                for (int t = 0; t < NT; ++t) { sL[t] = sigma[t]; sigma[t] = sR[t]; }
            }
        }
        for (; half >= 1; half >>= 1) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                ok[t] = off[t] + half < len[t];
                pos[t] = start[t] + off[t] + half;
            }
            score(pos, ok, s, sR);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (ROPE == 1) {
                    if (ok[t] && sR[t] > sL[t]) { off[t] += half; sL[t] = s[t]; sigma[t] = sR[t]; }
                } else if (ok[t] && s[t] > sigma[t]) { off[t] += half; sigma[t] = s[t]; }   // strict: tie keeps left
            }
        }
        // chunk score = max over the group's heads (waves)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int j = jt + t * 16 + n;
            if (kq == 0) sh_sigma[it & 1][wv][t * 16 + n] = sigma[t];
            if (a.out_rep != nullptr && kq == 0 && j < a.max_chunks) {
                const int64_t row = ((int64_t)(pr.b * a.ge.Hq + h) * a.ge.Mq + pr.m);
                a.out_rep[row * a.max_chunks + j] = valid[t] ? start[t] + off[t] : -1;
            }
        }
        __syncthreads();
        if (threadIdx.x < NT * 16) {
            const int j = jt + threadIdx.x;
            if (j < a.max_chunks) {
                float best = sh_sigma[it & 1][0][threadIdx.x];
                for (int g2 = 1; g2 < G; ++g2) best = fmaxf(best, sh_sigma[it & 1][g2][threadIdx.x]);
                if (part > 0) best = fmaxf(best, sh_best[it][threadIdx.x]);
                if (part + 1 < parts) {
                    sh_best[it][threadIdx.x] = best;
                } else {
                    // validity is the same for every head; recompute it for this slot
                    const bool v = slot_start(pr, a.parent_starts, a.n_parent, a.ratio_log2, a.chunk, p, j) >= 0;
                    a.out_scores[(int64_t)p * a.max_chunks + j] = v ? (KV8 ? best * a.k_scale : best) : -INFINITY;
                }
            }
        }
        // no barrier here: every wave has left its searches (the barrier above), the next chunk group
        // writes the other sh_sigma buffer, and sh_best is per chunk group
    }
    }
}

template <int MT, bool WIDE, int ROPE, bool PAGED, bool KV8 = false>
static void launch_prefill_w(const PruneArgs &a, int P, const RopeView &rope, hipStream_t st)
{
    constexpr int NT = 2;
    // several chunk groups per workgroup amortise the staging of the queries, as long as the
    // launch still has a few thousand workgroups
    int iters = kPrefillMaxIters;
    while (iters > 1 && (int64_t)P * ((a.max_chunks + NT * 16 * iters - 1) / (NT * 16 * iters)) < 2048) iters >>= 1;
    const int per_wg = NT * 16 * iters;
    dim3 grid(P, (a.max_chunks + per_wg - 1) / per_wg);
    KernelTimer timer(stage_name(kNamePrunePrefill, a.parent_starts == nullptr, a.chunk), st);
    switch (a.ge.G) {
    case 1: hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 1, WIDE, ROPE, PAGED, 1, KV8>), grid, dim3(64), 0, st, a, iters, rope); break;
    case 2: hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 2, WIDE, ROPE, PAGED, 1, KV8>), grid, dim3(128), 0, st, a, iters, rope); break;
    case 4:
        if constexpr (ROPE == 2 && MT == 4) {
            if ((int64_t)grid.x * grid.y <= 2ll * compute_units()) {
                hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 4, WIDE, ROPE, PAGED, 1, KV8, true>), grid, dim3(256), 0, st, a, iters, rope);
                break;
            }
        }
        hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 4, WIDE, ROPE, PAGED, 1, KV8>), grid, dim3(256), 0, st, a, iters, rope);
        break;
    default:
        // 8 heads with 64-query blocks: 8 waves of ~160 registers fit a CU once only, two passes of 4
        // waves fit three times; with RoPE the query operands alone take more registers than 8 waves
        // leave each other
        if constexpr (MT == 4)
            hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 4, WIDE, ROPE, PAGED, 2, KV8>), grid, dim3(256), 0, st, a, iters, rope);
        else
            hipLaunchKernelGGL((prune_prefill_kernel<MT, NT, 8, WIDE, ROPE, PAGED, 1, KV8>), grid, dim3(512), 0, st, a, iters, rope);
        break;
    }
}

}  // namespace ihip
