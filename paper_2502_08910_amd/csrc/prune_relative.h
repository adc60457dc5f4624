// Pruning-stage scoring for chunked prefill with relative-style dynamic RoPE (Sec. 4 "Dynamic RoPE for OOL
// generalization"; ApplyRopeQ / ApplyRopeK after Alg. 3): the kernel template and its launcher, shared by the bf16 and
// the E4M3 translation units.
//
// Every query of the block sits at n_stream+1, a left-branch key at 0, a right-branch key (and the representative in
// the chunk score) at 1.  With a table of true rotations the key rotations fold into the queries: two rotated copies of
// the query operands, q_L = R(n_stream+1) q and q_R = R(n_stream) q.  Each is kept as a bf16 value plus the
// bf16-rounded rest, and both are multiplied on the matrix cores, so that a score agrees with the product of the fp32
// rotations to about 2^-17 relative and a selection is decided as an fp32 evaluation decides it.
//
// Late scores.  A level's candidates are needed as right branches at once, as left branches only if they win: a winner
// is the left key of the next comparison (about one candidate in level + 1 wins).  And a first key's score as a right
// branch is needed only while it has not lost.  So a level multiplies its candidates with q_R alone; the columns that
// won are packed into as few 16-column products with q_L as they take, from the rows that are still in LDS, while the
// next level's rows are on their way.  A quarter of the matrix work of scoring every candidate as both.
//
// Mapping.  A wave walks the searches of 64 chunks at a time, one per lane: candidates are the columns of two
// v_mfma_f32_32x32x16_bf16 tiles, whose maxima over 32 queries end up in the lane of their chunk after one row swap
// (v_permlane32_swap of the two tiles' maxima).  What bounds this kernel is the chain of a search level (choose rows, fetch them,
// multiply, exchange maxima, decide) with only two waves per SIMD to cover it -- the four operand sets of 32 queries
// take 128 registers --, so a level is kept short and wide: one LDS round trip for each step of 64 searches, a
// handful of vector instructions to decide, and the two waves of a head share the candidate rows, each fetching half.
// First stage, 2,048 queries on 128K keys, chunks of 64, 32 heads: 898 us with every candidate scored both ways, 32
// chunks per wave and own copies of the rows; 850 us with late scores alone; 675 us this way.  E4M3 rows, 1,024 queries on 32K
// keys: 150 -> 116 us, in pages 151 -> 117 (48-80 bytes of scratch per lane).  Few workgroups walk 32 searches per wave (see
// launch_relative).  Two groups of 32 chunks in turn, one group's rows on their way while the other's are
// multiplied, were no faster than one (850): twice the LDS round trips.
//
// Two waves per query head, 32 queries each.  They fetch half of a level's candidate rows each into a tile of the head and
// exchange their maxima over the queries through LDS.  Both are handshakes of the two waves, not workgroup barriers
// (which would put all waves of the workgroup in step): a wave does its part, raises its turn counter (LDS keeps a
// wave's requests in order) and goes on once the other's counter has reached the same turn.  Both raise before they
// wait and both are resident (one workgroup), so the wait ends; it is bounded all the same.  Two tiles per head: rows of
// the next level land in one while late scores read the other.  Blocks of 16 and 32 queries need one wave per head and
// run in prune_prefill_kernel.
#pragma once

#include "prune_prefill.h"

namespace ihip {

// COLS: searches of a wave, 64 or 32 (lanes 32.. then walk the same searches as lanes 0..31)
// PARTS, WIDE, PAGED, KV8: as in prune_prefill_kernel
template <int COLS, int G, bool WIDE, bool PAGED, int PARTS, bool KV8>
__global__ __launch_bounds__(128 * G, 2) void prune_relative_kernel(const PruneArgs a, const int iters, const RopeView rope)
{
    static_assert(!PAGED || WIDE, "paged pools are addressed with 64-bit offsets");
    constexpr int QS = 2;                            // waves of a head
    static_assert(COLS == 64 || COLS == 32, "one search per lane, or one per two");
    constexpr int kCols = COLS;
    constexpr int NWV = G * QS;                      // waves of the workgroup
    constexpr int MTW = 2;                           // 16-query tiles of a wave
    constexpr int kTile = kCols * kD;                // rows of 256 bytes, no padding
    constexpr int kBufs = 2;                         // tiles of a head
    constexpr int kTiles = G * kBufs;
    constexpr int kLoads = kCols / 4 / QS;           // four-row loads of a level that are this wave's
    constexpr uint32_t kFourRows = 4 * kD * 2, kTileBytes = kTile * 2;
    using raw_t = typename std::conditional<KV8, uint2, uint4>::type;         // a lane's 8 elements of a row as fetched
    using off_t = typename std::conditional<WIDE, int64_t, uint32_t>::type;   // byte (WIDE: element) offset of a row
    __shared__ float sh_sigma[2][G][kCols];          // two buffers: an iteration writes while the last one is still read
    __shared__ float sh_best[kPrefillMaxIters / 2][kCols];      // chunk scores over the head parts done so far
    // a wave's maxima over its queries, by column: [0] of a level's candidates as right branches, [1] of the keys that won
    // the level before as left branches, [2] of first keys that are still ahead as right branches.  Two buffers: the
    // late ones of the next exchange are written while the partner may still read the last ones.
    __shared__ float sh_max[2][NWV][3][kCols];
    __shared__ uint8_t sh_list[NWV][kCols];          // columns that need a late score, packed
    __shared__ uint32_t sh_turn[NWV];
    // tile b of head h at (h * kBufs + b) * kTile; first the rows that all waves share: tile 0 first keys, tile 1 first keys
    // of the right halves
    __shared__ __attribute__((aligned(16))) uint16_t sh_rows[kTiles * kTile];
    // KV head fastest, as in prune_prefill_kernel
    const int p = ((blockIdx.x / a.ge.Hkv / a.ge.Mq) * a.ge.Hkv + blockIdx.x % a.ge.Hkv) * a.ge.Mq +
                  (blockIdx.x / a.ge.Hkv) % a.ge.Mq;
    const Problem pr = problem_of(a.ge, p);
    const int lane = threadIdx.x & 63, col = lane & (kCols - 1), wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hh = wv / QS, qs = wv % QS;            // the wave's query head of the group, and its share of the queries
    if (lane == 0) sh_turn[wv] = 0;                  // a workgroup barrier follows before the first handshake
    const int n16 = lane & 15, kq = lane >> 4;       // 16x16x32 operands: row / column and group of 8 dims
    const int n32 = lane & 31, kh = lane >> 5;       // 32x32x16 operands
    int h = pr.g * (G * PARTS) + hh;

    const uint16_t *kb = PAGED ? a.k + pr.g * a.k_sh : a.k + pr.b * a.k_sb + pr.g * a.k_sh;
    const int32_t *table = PAGED ? a.paged.block_table + (int64_t)pr.b * a.paged.table_stride : nullptr;
    // offset of key row `pos` from kb: bytes (one full-rate 24-bit multiply), WIDE: elements
    auto row_at = [&](int pos) -> off_t {
        if constexpr (PAGED)
            return (int64_t)table[pos >> a.paged.page_log2] * a.k_sb + (int64_t)(pos & ((1 << a.paged.page_log2) - 1)) * a.k_st;
        else if constexpr (WIDE) return (int64_t)pos * a.k_st;
        else return __umul24((uint32_t)pos, (uint32_t)a.k_st * 2u);
    };
    // Four-row loads: lanes 16*kq..+15 fetch one whole row each, 16 (E4M3: 8) bytes per lane, straight into LDS at
    // dst + lane*16; piece c of tile row R sits in slot c ^ (R%16) (applied on the source side), so that the rows of an
    // operand read hit different bank groups.  swz = R%16 of this lane's row.  Written as assembly, as in prune_prefill_kernel.
    auto load4 = [&](off_t at, uint32_t dst, int swz) {
        if constexpr (WIDE) global_to_lds(dst, kb + at + ((n16 ^ swz) << 3));
        else global_to_lds(dst, kb, at + (uint32_t)((n16 ^ swz) << 4));
    };
    // E4M3 (always WIDE): through registers, widened on the way
    auto fetch = [&](off_t at, int swz) { return *reinterpret_cast<const raw_t *>(kb + at + (n16 ^ swz) * (int)(sizeof(raw_t) / 2)); };
    auto put16 = [&](uint16_t *four_rows, const uint4 piece) { *reinterpret_cast<uint4 *>(four_rows + kq * kD + n16 * 8) = piece; };
    auto lds_addr = [&](const uint16_t *ptr) {
        return (uint32_t)__builtin_amdgcn_readfirstlane(
            (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)ptr);
    };
    auto from_lane = [&](off_t x, int src) -> off_t { return __shfl(x, src, 64); };

    uint16_t *head_tile = &sh_rows[hh * kBufs * kTile];
    const uint32_t dst_head = lds_addr(head_tile);

    // The rotated queries, value and rest: q_R as 32x32x16 operands, q_L as 16x16x32 operands
    bf16x8 qR[8], qRlo[8], qL[MTW][4], qLlo[MTW][4];
    auto load_queries = [&]() {
        int l = lane;                         // opaque: the addresses are formed here, not carried over the passes
        asm volatile("" : "+v"(l));
        const int n16 = l & 15, kq = l >> 4, n32 = l & 31, kh = l >> 5;
        const uint16_t *qb = a.q + pr.b * a.q_sb + (int64_t)h * a.q_sh + (int64_t)(pr.m * a.ge.b_q + qs * MTW * 16) * a.q_st;
        const float *c = rope.cos + (int64_t)a.ge.n_stream * (kD / 2), *sn = rope.sin + (int64_t)a.ge.n_stream * (kD / 2);
        // a set's pieces and their table rows are all requested before the first is turned
        {
            bf16x8 q[8];
            float4 tc[8], ts[8];
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const int piece = ks * 2 + kh;
                q[ks] = *reinterpret_cast<const bf16x8 *>(qb + (int64_t)n32 * a.q_st + piece * 8);
                tc[ks] = *reinterpret_cast<const float4 *>(c + piece * 4);
                ts[ks] = *reinterpret_cast<const float4 *>(sn + piece * 4);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) rotate_operand_split(q[ks], tc[ks], ts[ks], qR[ks], qRlo[ks]);
        }
        __builtin_amdgcn_sched_barrier(0);
        {
            bf16x8 q[MTW][4];
            float4 tc[4], ts[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int piece = ks * 4 + kq;
                tc[ks] = *reinterpret_cast<const float4 *>(c + kD / 2 + piece * 4);
                ts[ks] = *reinterpret_cast<const float4 *>(sn + kD / 2 + piece * 4);
#pragma unroll
                for (int mt = 0; mt < MTW; ++mt)
                    q[mt][ks] = *reinterpret_cast<const bf16x8 *>(qb + (int64_t)(mt * 16 + n16) * a.q_st + piece * 8);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) rotate_operand_split(q[mt][ks], tc[ks], ts[ks], qL[mt][ks], qLlo[mt][ks]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Scores of tile row `row` (this lane's column, of 32) as a right branch: maximum over half of this wave's queries,
    // the other half's is in lane ^ 32
    auto right_half = [&](const uint16_t *src, int row) {
        bf16x8 kr[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            kr[ks] = *reinterpret_cast<const bf16x8 *>(&src[row * kD + (((ks << 1) + kh) ^ (row & 15)) * 8]);
        f32x16 c;
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qRlo[ks], kr[ks], c, 0, 0, 0);   // the small terms first
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qR[ks], kr[ks], c, 0, 0, 0);
        float best = c[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) best = fmaxf(best, c[r]);
        return best;
    };
    // the maxima of two products (columns 0..31 and 32..63, or the same 32 twice), each lane its own column's
    auto both_halves = [&](float x0, float x1) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
        return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    };
    auto right_scores = [&](const uint16_t *src) {
        const float x0 = right_half(src, n32);
        if constexpr (kCols == 32) return both_halves(x0, x0);
        const float x1 = right_half(src, 32 + n32);
        return both_halves(x0, x1);
    };
    // Score of tile row `row` (this lane's column, of 16) as a left branch, maximum over this wave's queries
    auto left_score = [&](const uint16_t *src, int row) {
        bf16x8 kr[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            kr[ks] = *reinterpret_cast<const bf16x8 *>(&src[row * kD + (((ks << 2) + kq) ^ (row & 15)) * 8]);
        float best = -INFINITY;
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qLlo[mt][ks], kr[ks], c, 0, 0, 0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qL[mt][ks], kr[ks], c, 0, 0, 0);
            best = fmaxf(best, fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
        }
        return max_over_rows(best);
    };
    // the columns whose lane has `need` set, packed: sh_list[0..count)
    auto pack = [&](bool need) {
        need = need && lane < kCols;
        const uint64_t mask = __ballot(need);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (need) sh_list[wv][rank] = (uint8_t)lane;
        asm volatile("" ::: "memory");        // lanes read what other lanes of the wave wrote (LDS keeps the order)
        return (int)__popcll(mask);
    };
    auto late_left = [&](const uint16_t *src, bool need, float *out) {
        const int cnt = pack(need);
#pragma unroll 1
        for (int at = 0; at < cnt; at += 16) {
            const int c = at + n16 < cnt ? sh_list[wv][at + n16] : n16;
            const float v = left_score(src, c);
            if (kq == 0 && at + n16 < cnt) out[c] = v;
        }
        asm volatile("" ::: "memory");        // the list is written again only after it has been read
    };
    auto late_right = [&](const uint16_t *src, bool need, float *out) {
        const int cnt = pack(need);
#pragma unroll 1
        for (int at = 0; at < cnt; at += 32) {
            const int c = at + n32 < cnt ? sh_list[wv][at + n32] : n32;
            const float x = right_half(src, c);
            const float v = both_halves(x, x);
            if (kh == 0 && at + n32 < cnt) out[c] = v;
        }
        asm volatile("" ::: "memory");
    };
    uint32_t turn = 0;
    auto handshake = [&]() {                  // what this wave wrote to LDS before is there for its partner, and the other way round
        asm volatile("" ::: "memory");
        ++turn;
        if (lane == 0) __hip_atomic_store(&sh_turn[wv], turn, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        int budget = 1 << 18;                 // a wait is a few dozen turns of this loop; the bound is ~10 ms
        while ((int32_t)(__hip_atomic_load(&sh_turn[wv ^ 1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) - turn) < 0 &&
               --budget > 0)
            __builtin_amdgcn_s_sleep(1);
    };
    int xbuf = 0;                             // buffer of the next exchange
    // maximum of kind `what` for this lane's column in the last exchange, over all the block's queries
    auto exchanged = [&](int what) {
        return fmaxf(sh_max[xbuf ^ 1][wv][what][col], sh_max[xbuf ^ 1][wv ^ 1][what][col]);
    };
    auto exchange = [&](float right) {        // -> the right-branch maximum; the late ones of this turn can be read
        sh_max[xbuf][wv][0][col] = right;
        handshake();
        xbuf ^= 1;
        return fmaxf(right, sh_max[xbuf ^ 1][wv ^ 1][0][col]);
    };

    if constexpr (PARTS == 1) load_queries();
#pragma unroll 1
    for (int part = 0; part < PARTS; ++part) {
    if constexpr (PARTS > 1) {
        h = pr.g * (G * PARTS) + part * G + hh;
        load_queries();
    }
#pragma unroll 1
    for (int it = 0; it < iters; ++it) {
        const int jt = (blockIdx.y * iters + it) * kCols;
        if (jt >= a.max_chunks) break;               // the whole workgroup
        const int j = jt + col;
        const int start = j < a.max_chunks ? slot_start(pr, a.parent_starts, a.n_parent, a.ratio_log2, a.chunk, p, j) : -1;
        const int len = start >= 0 ? min(a.chunk, pr.hi - start) : 0;
        int off = 0, half = a.chunk >> 1;
        // The first key of a chunk and of its right half are the same rows for every head of the group: fetched once, the
        // four-row loads dealt to the waves.
        {
            constexpr int kOfTile = kCols / 4, kPerWave = 2 * kOfTile / NWV;
            static_assert(kPerWave * NWV == 2 * kOfTile, "the wave count divides the loads");
            const off_t at0 = row_at(max(start, 0)), at1 = row_at(half >= 1 && half < len ? start + half : 0);
            raw_t raw[KV8 ? kPerWave : 1];
#pragma unroll
            for (int i = 0; i < kPerWave; ++i) {
                const int ld = wv * kPerWave + i, r = ld % kOfTile;  // wave-uniform
                const off_t at = from_lane(ld < kOfTile ? at0 : at1, r * 4 + kq);
                if constexpr (KV8) raw[i] = fetch(at, (r & 3) * 4 + kq);
                else load4(at, lds_addr(sh_rows) + ld * kFourRows, (r & 3) * 4 + kq);
            }
            if constexpr (KV8) {
#pragma unroll
                for (int i = 0; i < kPerWave; ++i) put16(&sh_rows[(wv * kPerWave + i) * 4 * kD], fp8x8_to_bf16x8(raw[KV8 ? i : 0]));
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        }
        __syncthreads();

        // candidates of a level on their way to tile b of the head: rows at start + off + half (row 0 where the search
        // has ended); this wave's share of them
        raw_t raw[KV8 ? kLoads : 1];
        auto request = [&](int half, int b) {
            const off_t at = row_at(off + half < len ? start + off + half : 0);
            off_t cand[kLoads];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) cand[i] = from_lane(at, (qs * kLoads + i) * 4 + kq);
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                if constexpr (KV8) raw[i] = fetch(cand[i], (i & 3) * 4 + kq);
                else load4(cand[i], dst_head + b * kTileBytes + (qs * kLoads + i) * kFourRows, (i & 3) * 4 + kq);
            }
        };
        auto landed = [&](int b) {
            if constexpr (KV8) {
#pragma unroll
                for (int i = 0; i < kLoads; ++i)
                {
                    put16(head_tile + b * kTile + (qs * kLoads + i) * 4 * kD, fp8x8_to_bf16x8(raw[KV8 ? i : 0]));
                    __builtin_amdgcn_sched_barrier(0);           // one row group after the other: registers
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            handshake();
        };

        // first comparison: first keys as left branches, first keys of the right halves as right branches
        float l0;
        {
            float l[kCols / 16];
#pragma unroll
            for (int t = 0; t < kCols / 16; ++t) {
                l[t] = left_score(&sh_rows[0], t * 16 + n16);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (kCols == 32) l0 = (kq & 1) == 0 ? l[0] : l[1];
            else l0 = kq == 0 ? l[0] : kq == 1 ? l[1] : kq == 2 ? l[2] : l[3];
        }
        sh_max[xbuf][wv][1][col] = l0;
        // sL: the current left key as a left branch; sigma: the same key as a right branch, which is what the chunk score
        // takes.  `won`: sL is still to come (the key won the last level); `ahead`: sigma is (the first key has not lost).
        float sigma = exchange(right_scores(&sh_rows[kTile]));
        float sL = exchanged(1);
        bool won = half >= 1 && half < len && sigma > sL;        // strict: tie keeps left
        bool ahead = !won;
        off = won ? half : 0;
        late_right(&sh_rows[0], ahead, sh_max[xbuf][wv][2]);
        if (half > 1) late_left(&sh_rows[kTile], won, sh_max[xbuf][wv][1]);
        half >>= 1;
        if (half >= 1) {
            __syncthreads();                         // every wave is done with the shared tiles: they are their heads' again
            request(half, 0);
        }
        bool levels = false;
        for (int b = 0; half >= 1; half >>= 1, b ^= 1) {
            landed(b);
            const uint16_t *rows = head_tile + b * kTile;
            const float right = exchange(right_scores(rows));
            sL = won ? exchanged(1) : sL;
            if (!levels) sigma = ahead ? exchanged(2) : sigma;
            levels = true;
            won = off + half < len && right > sL;                // strict: tie keeps left
            off += won ? half : 0;
            sigma = won ? right : sigma;
            if (half > 1) {
                request(half >> 1, b ^ 1);
                late_left(rows, won, sh_max[xbuf][wv][1]);
            }
        }
        if (!levels) {                               // chunks of one or two keys: no level has picked these up
            (void)exchange(0.f);
            sigma = ahead ? exchanged(2) : sigma;
        }
        // chunk score = max over the group's heads (waves)
        if (qs == 0) {
            sh_sigma[it & 1][hh][col] = sigma;
            if (a.out_rep != nullptr && lane < kCols && j < a.max_chunks) {
                const int64_t row = ((int64_t)(pr.b * a.ge.Hq + h) * a.ge.Mq + pr.m);
                a.out_rep[row * a.max_chunks + j] = start >= 0 ? start + off : -1;
            }
        }
        __syncthreads();
        if (wv == 0 && lane < kCols && j < a.max_chunks) {
            float best = sh_sigma[it & 1][0][col];
            for (int g2 = 1; g2 < G; ++g2) best = fmaxf(best, sh_sigma[it & 1][g2][col]);
            if (part > 0) best = fmaxf(best, sh_best[it][col]);
            if (part + 1 < PARTS) sh_best[it][col] = best;
            else a.out_scores[(int64_t)p * a.max_chunks + j] = start >= 0 ? (KV8 ? best * a.k_scale : best) : -INFINITY;
        }
        // no barrier here: every wave has left its searches (the barrier above), the next iteration writes the other
        // sh_sigma buffer, and sh_best is per iteration and only this wave's
    }
    }
}

// 64-query blocks
template <int COLS, bool WIDE, bool PAGED, bool KV8>
static void launch_relative_c(const PruneArgs &a, int P, const RopeView &rope, hipStream_t st)
{
    // several iterations per workgroup amortise the rotation of the queries, as long as the launch still has
    // a few thousand workgroups
    int iters = COLS == 32 ? 1 : kPrefillMaxIters / 2;
    while (iters > 1 && (int64_t)P * ((a.max_chunks + COLS * iters - 1) / (COLS * iters)) < 2048) iters >>= 1;
    const int per_wg = COLS * iters;
    dim3 grid(P, (a.max_chunks + per_wg - 1) / per_wg);
    KernelTimer timer(stage_name(kNamePrunePrefill, a.parent_starts == nullptr, a.chunk), st);
    switch (a.ge.G) {
    case 1: hipLaunchKernelGGL((prune_relative_kernel<COLS, 1, WIDE, PAGED, 1, KV8>), grid, dim3(128), 0, st, a, iters, rope); break;
    case 2: hipLaunchKernelGGL((prune_relative_kernel<COLS, 2, WIDE, PAGED, 1, KV8>), grid, dim3(256), 0, st, a, iters, rope); break;
    case 4: hipLaunchKernelGGL((prune_relative_kernel<COLS, 4, WIDE, PAGED, 1, KV8>), grid, dim3(512), 0, st, a, iters, rope); break;
    default:                                         // 8 heads: two passes of 4
        hipLaunchKernelGGL((prune_relative_kernel<COLS, 4, WIDE, PAGED, 2, KV8>), grid, dim3(512), 0, st, a, iters, rope);
        break;
    }
}

template <bool WIDE, bool PAGED, bool KV8>
static void launch_relative(const PruneArgs &a, int P, const RopeView &rope, hipStream_t st)
{
    // While the workgroups of 32 searches all run at once (eight waves of 256 registers fill a compute unit, two leave room for
    // four of them), half the products per level make the shorter chain: 64 queries, 32 heads, chunks of 64, 16K keys 24.1 us
    // with 64 searches per wave, 18.1 with 32; 64K keys (256 workgroups) 24.4 and 18.8.  Beyond, 64 do more per row:
    // 128K keys 27.0 and 36.2.  One head per group, chunks of 64, 1,024 workgroups 20.9 and 18.7, chunks of 4, 936 of them
    // 12.8 and 13.5; two heads, 512, 18.8 and 19.2.
    const int per_cu = a.ge.G > 1 ? 1 : a.chunk >= 16 ? 4 : 2;
    const bool few = (int64_t)P * ((a.max_chunks + 31) / 32) <= (int64_t)per_cu * compute_units();
    if (few) launch_relative_c<32, WIDE, PAGED, KV8>(a, P, rope, st);
    else launch_relative_c<64, WIDE, PAGED, KV8>(a, P, rope, st);
}

// Relative-style RoPE: 64-query blocks have a kernel of their own, smaller blocks (whose rotated operand sets fit one wave
// per head, with two waves per SIMD) take the general one: 32 queries 105 us against 98 there but 30 against 38 with one
// head per group, 16 queries 115 against 155 (1,024 queries on 32K keys).
template <int MT, bool WIDE, bool PAGED, bool KV8 = false>
static void launch_relative_w(const PruneArgs &a, int P, const RopeView &rope, hipStream_t st)
{
    if constexpr (MT == 4) launch_relative<WIDE, PAGED, KV8>(a, P, rope, st);
    else launch_prefill_w<MT, WIDE, 1, PAGED, KV8>(a, P, rope, st);
}

}  // namespace ihip
