// Decode pruning stage on the matrix cores (b_q == 1): Alg. 3's search and Alg. 2's chunk score, K from device memory
// (strides or pages) or behind the host tier, without RoPE or with the relative style.  One query per head makes this a gather, not a contraction: what
// it cannot do without are the rows.  The matrix cores take the arithmetic off the vector ALUs: 16 gathered rows
// against 16 query columns is four v_mfma_f32_16x16x32_bf16 (E4M3 rows are widened, exact), of whose 256 products the 16
// that are wanted are picked in the registers; the vector form needs some 30 instructions for every four rows (45 with
// two rotated queries), and with 128-byte rows or two rotated queries those, not the rows, were the time.
//
// A wave walks 64 searches, one per lane: 64/G chunks x G heads, in four 16-row tiles (host tier: 16 searches, one tile).  Tile t, row r = 4*kq + i is owned
// by lane (kq, n = 4t + i): the product's column n, rows 4*kq..+3 are in that lane's accumulator, so with column n
// holding the query of head n % G the owner finds its own score in register n % 4 -- no value crosses lanes except the
// row offsets, handed from the owners to the lanes of their row group (register broadcasts within 16 lanes).
//
// Rows are fetched whole, by neighbouring lanes, and reach operand layout through LDS.  Fetched in operand layout a load names 16 rows
// at once, 16 bytes of each to a lane whose neighbour wants another row: 64 look-ups in the L1 instead of 16 (8 with E4M3 rows), which was
// the time of a search level.  Four sequences of 250K keys in E4M3 pages with relative RoPE, operand layout / whole rows (us): stages of
// 256, 64, 16 and 4 keys 25.3 / 22.3, 20.0 / 17.3, 13.9 / 12.8, 13.8 / 11.8; one pass over 8K keys (prune_decode_nest.h) 5.7 / 4.8.
// Relative style (see prune_relative.h): columns 0..7 hold q_L, 8..15 q_R; the two halves are exchanged by one row rotation.
// The rotated queries are fp32, kept as three bf16 operands (value, rest, rest of the rest: 24 bits and more), so that a score is as
// good as an fp32 one.
//
// Operand layout: lane (n, kq) holds 8 dims of row or column n; any assignment of dims to (step, kq) serves as long as both
// sides agree.  bf16 rows: step ks, dims 32*ks + 8*kq.. (one 16-byte piece).  E4M3 rows: piece j brings dims 64*j + 16*kq..+15,
// steps 2j and 2j+1.
#pragma once

#include "prune_prefill.h"

namespace ihip {

// The query operands of a lane: column n16's head, 8 dims of group kq per step, PARTS bf16 operands each (1: the query as
// it is; 3: rotated by table row `pos`, fp32 in three parts)
template <bool KV8, int PARTS>
__device__ inline void decode_query_operands(const uint16_t *q_row, int kq, const RopeView &rope, int pos, bf16x8 (&q)[PARTS][4])
{
    uint4 w[4];
    float4 c[PARTS > 1 ? 4 : 1], s[PARTS > 1 ? 4 : 1];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int d0 = KV8 ? (ks >> 1) * 64 + kq * 16 + (ks & 1) * 8 : ks * 32 + kq * 8;
        w[ks] = *reinterpret_cast<const uint4 *>(q_row + d0);
        if constexpr (PARTS > 1) {
            c[ks] = *reinterpret_cast<const float4 *>(rope.cos + (int64_t)pos * (kD / 2) + d0 / 2);
            s[ks] = *reinterpret_cast<const float4 *>(rope.sin + (int64_t)pos * (kD / 2) + d0 / 2);
        }
    }
    if constexpr (PARTS > 1) __builtin_amdgcn_sched_barrier(0);      // everything is requested before anything is turned
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        if constexpr (PARTS == 1) {
            q[0][ks] = __builtin_bit_cast(bf16x8, w[ks]);
        } else {
            float x[8], y[8];
            unpack8(w[ks], x);
            const float cc[4] = {c[ks].x, c[ks].y, c[ks].z, c[ks].w}, ss[4] = {s[ks].x, s[ks].y, s[ks].z, s[ks].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                y[2 * i] = x[2 * i] * cc[i] - x[2 * i + 1] * ss[i];
                y[2 * i + 1] = x[2 * i] * ss[i] + x[2 * i + 1] * cc[i];
            }
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
                uint32_t u[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    u[i] = pack_bf16x2(y[2 * i], y[2 * i + 1]);
                    y[2 * i] -= __uint_as_float(u[i] << 16);              // exact
                    y[2 * i + 1] -= __uint_as_float(u[i] & 0xffff0000u);
                }
                q[part][ks] = __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
            }
        }
    }
}

// 16 rows x 16 columns; raw: this lane's pieces of row n16 (bf16: one per step, E4M3: one per two steps)
template <bool KV8, int PARTS>
__device__ inline f32x4 decode_products(const uint4 (&raw)[KV8 ? 2 : 4], const bf16x8 (&q)[PARTS][4])
{
    bf16x8 k[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        if constexpr (KV8) {
            const uint4 w = raw[ks >> 1];
            k[ks] = __builtin_bit_cast(bf16x8, fp8x8_to_bf16x8((ks & 1) ? make_uint2(w.z, w.w) : make_uint2(w.x, w.y)));
        } else {
            k[ks] = __builtin_bit_cast(bf16x8, raw[KV8 ? 0 : ks]);
        }
    }
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int part = PARTS - 1; part >= 0; --part)        // the small terms first
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[ks], q[part][ks], c, 0, 0, 0);
    return c;
}

__device__ inline float pick4(const f32x4 c, int i)      // c[i], in registers
{
    const float a = (i & 1) ? c[1] : c[0], b = (i & 1) ? c[3] : c[2];
    return (i & 2) ? b : a;
}
__device__ inline float row_ror8(float v) { return dpp_f32<0x128>(v); }
// lane N of each row of 16, in all its lanes
template <int N>
__device__ inline int row_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xf, 0xf, true); }
template <int N>
__device__ inline uint32_t row_lane(uint32_t v) { return (uint32_t)row_lane<N>((int)v); }
template <int N>
__device__ inline int64_t row_lane(int64_t v)
{
    return (int64_t)(((uint64_t)row_lane<N>((uint32_t)(v >> 32)) << 32) | row_lane<N>((uint32_t)v));
}
template <int N, class F>
__device__ inline void for_each_tile(F f)                // f(0), ..., f(N - 1), each a constant
{
    if constexpr (N > 0) {
        for_each_tile<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}
__device__ inline float other_quad(float v) { return dpp_f32<0x1B>(dpp_f32<0x141>(v)); }   // lane n ^ 4 of a row: half mirror, then each quad reversed

// Where the rows of (sequence, KV head) are, and how a lane's row offset is formed and handed round.  NARROW: byte offsets of 32 bits
// from a scalar base (every row of the slab within 4 GB); otherwise elements in 64 bits; SRC 2: pages.
template <int SRC, bool NARROW>
struct DecodeRows {
    const uint16_t *kb;
    const int32_t *table;
    int64_t k_sb, k_st;
    int page_log2;
    using off_t = typename std::conditional<NARROW, uint32_t, int64_t>::type;
    __device__ DecodeRows(const PruneArgs &a, const Problem &pr)
    {
        kb = SRC == 2 ? a.k + pr.g * a.k_sh : a.k + pr.b * a.k_sb + pr.g * a.k_sh;
        table = SRC == 2 ? a.paged.block_table + (int64_t)pr.b * a.paged.table_stride : nullptr;
        k_sb = a.k_sb;
        k_st = a.k_st;
        page_log2 = a.paged.page_log2;
    }
    __device__ off_t at(int pos, int page) const         // page: of a paged pool
    {
        if constexpr (SRC == 2) return (int64_t)page * k_sb + (int64_t)(pos & ((1 << page_log2) - 1)) * k_st;
        else if constexpr (NARROW) return (uint32_t)pos * (uint32_t)(k_st * 2);
        else return (int64_t)pos * k_st;
    }
    // 16 bytes at byte `b` of the row at `off`
    __device__ uint4 load(off_t off, int b) const
    {
        if constexpr (NARROW) return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(kb) + (uint64_t)(off + (uint32_t)b));
        else return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(kb + off) + b);
    }
};

// SRC 1: rows of the host tier.  A lane's "offset" is the row's address, so that each owner looks its row up, and notes it, once; position
// -1 (nothing may be noted): a row of the query, which is there
template <>
struct DecodeRows<1, false> {
    CachedRows src;
    const uint16_t *unread;
    using off_t = int64_t;
    __device__ DecodeRows(const PruneArgs &a, const Problem &pr) : src(KeySource<1>::make(a, pr)), unread(a.q + pr.b * a.q_sb) {}
    // slot: slot_of(max(pos, 0)), whose load several rows may wait for together
    __device__ off_t at(int pos, int slot) const { return (int64_t)(uintptr_t)(pos >= 0 ? src.row(pos, true, slot) : unread); }
    __device__ uint4 load(off_t off, int b) const      // named as global memory, which the compiler cannot tell of an address
    {
        typedef uint32_t words __attribute__((ext_vector_type(4)));
        return __builtin_bit_cast(uint4, *(const __attribute__((address_space(1))) words *)((uintptr_t)off + b));
    }
};

// The 16 rows of tile T on their way: row 4 * kq + i, whole, by the lanes of row group kq, whose lane 4 * T + i has its offset in `off`.
// (All lanes take part: a lane that is switched off hands out zero.)
template <int T, bool KV8, class Rows>
__device__ inline void request_tile(const Rows &rows, typename Rows::off_t off, int n, uint4 (&raw)[KV8 ? 2 : 4])
{
    const auto at0 = row_lane<4 * T>(off), at1 = row_lane<4 * T + 1>(off), at2 = row_lane<4 * T + 2>(off), at3 = row_lane<4 * T + 3>(off);
    if constexpr (KV8) {
        raw[0] = rows.load(n < 8 ? at0 : at1, (n & 7) * 16);
        raw[1] = rows.load(n < 8 ? at2 : at3, (n & 7) * 16);
    } else {
        raw[0] = rows.load(at0, n * 16);
        raw[1] = rows.load(at1, n * 16);
        raw[2] = rows.load(at2, n * 16);
        raw[3] = rows.load(at3, n * 16);
    }
}
// ... and into operand layout through `tile`, 16 rows of the wave's own in LDS
template <bool KV8>
__device__ inline void arrange_tile(uint4 *tile, int n, int kq, uint4 (&raw)[KV8 ? 2 : 4])
{
    constexpr int kLoads = KV8 ? 2 : 4, kPieces = KV8 ? 8 : 16;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int r = 4 * kq + (KV8 ? 2 * i + (n >> 3) : i);
        tile[r * kPieces + ((n ^ r) & (kPieces - 1))] = raw[i];           // piece c of row r at c ^ r
    }
    asm volatile("" ::: "memory");            // lanes read what other lanes of the wave wrote (LDS keeps the order)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) raw[i] = tile[n * kPieces + (((i * 4 + kq) ^ n) & (kPieces - 1))];
    asm volatile("" ::: "memory");
}
constexpr int decode_row_pieces(bool fp8) { return fp8 ? 8 : 16; }

// What a wave without a single chunk writes for its n <= 64 slots j0..
template <int G>
__device__ inline void write_no_chunks(const PruneArgs &a, const Problem &pr, int p, int j0, int n)
{
    const int i = threadIdx.x & 63, j = j0 + i;
    if (i >= n || j >= a.max_chunks) return;
    a.out_scores[(int64_t)p * a.max_chunks + j] = -INFINITY;
    if (a.out_rep == nullptr) return;
    for (int h = 0; h < G; ++h) {
        const int64_t row = (int64_t)(pr.b * a.ge.Hq + pr.g * G + h) * a.ge.Mq + pr.m;
        a.out_rep[row * a.max_chunks + j] = -1;
    }
}

// Tiles of a wave.  Host tier: one, whose 16 owners look their rows up in the bank and hand them to the lanes of their row group; four times
// the waves (8K to 32K keys all in the banks, 64 heads on 8, bf16: 100 -> 80 us a layer, 32 on 8 86 -> 76).  Vector kernel / this one
// (us): 8K bf16 keys, 32 heads on 8, banks that hold few of them 291 / 273, all 68 / 58, 500K E4M3 with RoPE 64 on 8 all 278 / 219;
// one head a group is where it loses, up to 5 us of 50 (4K to 12K keys in the banks), a layer of four stages on 17K keys 96 / 108; it
// is taken there too, for the bits that contiguous rows give.
constexpr int decode_search_tiles(int src) { return src == 1 ? 1 : 4; }

constexpr int kDecodePages = 16;              // page ids of a chunk kept in LDS; further ones are looked up in the table

// Eight heads over bf16 pages with rotated queries: left alone the compiler takes 172 registers, two waves per SIMD; told to
// leave room for three it takes 124 (28 sequences of 100K keys: a layer 756 -> 685 us).  The same for chunks of four below: 90
// instead of 96-100, five waves instead of four.
template <int G, bool ROPE, int SRC, bool KV8, bool NARROW>
__global__ __launch_bounds__(256, G == 8 && ROPE && SRC == 2 && !KV8 ? 3 : 1) void prune_decode_tile_kernel(const PruneArgs a, const RopeView rope)
{
    static_assert(SRC == 0 || !NARROW, "paged pools and the host tier are addressed with 64-bit offsets");
    constexpr int PARTS = ROPE ? 3 : 1;
    constexpr int NT = decode_search_tiles(SRC);
    constexpr int kPerTile = 16 / G;          // chunks of a tile
    constexpr int kChunks = NT * kPerTile;    // chunks of a wave
    constexpr int kLoads = KV8 ? 2 : 4;
    using Rows = DecodeRows<SRC, NARROW>;
    using off_t = typename Rows::off_t;
    __shared__ int32_t sh_pages[SRC == 2 ? 4 * kChunks * kDecodePages : 1];
    __shared__ uint4 sh_rows[kDecodeTileWaves * 16 * decode_row_pieces(KV8)];
    const int p = a.grid.problem();
    const Problem pr = problem_of(a.ge, p);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4, quad = n >> 2;
    const int j0 = (a.grid.part() * (blockDim.x >> 6) + wv) * kChunks;
    if (j0 >= a.max_chunks) return;

    // this lane's search: chunk `ci` of the wave, head `hd` of the group
    const int r = 4 * kq + (n & 3);
    const int ci = quad * kPerTile + r / G, hd = r % G;
    const int j = j0 + ci;
    const bool owner = quad < NT;             // of a search
    const int start = owner && j < a.max_chunks ? slot_start(pr, a.parent_starts, a.n_parent, a.ratio_log2, a.chunk, p, j) : -1;
    const bool valid = start >= 0;
    const int len = valid ? min(a.chunk, pr.hi - start) : 0;
    // No chunk at all (a sequence that ends before its middle range, an idle place of the batch, the tail of a short list):
    // nothing may be read.  Where the wave has a chunk, lanes without one read key 0 of the sequence: it is there, since a
    // chunk starts below pr.hi <= its length.
    if (__ballot(valid) == 0) {
        write_no_chunks<G>(a, pr, p, j0, kChunks);
        return;
    }

    bf16x8 q[PARTS][4];
    {
        const int qh = G == 8 ? (n & 7) : n % G;
        const uint16_t *qb = a.q + pr.b * a.q_sb + (int64_t)(pr.g * G + qh) * a.q_sh + (int64_t)pr.m * a.q_st;
        decode_query_operands<KV8, PARTS>(qb, kq, rope, a.ge.n_stream + (n < 8 ? 1 : 0), q);
    }
    const Rows rows(a, pr);
    const int base = SRC == 1 ? start : max(start, 0);
    const int unread = SRC == 1 ? -1 : base;  // position for a lane that needs no row
    int32_t *pages = &sh_pages[SRC == 2 ? wv * kChunks * kDecodePages : 0];
    if constexpr (SRC == 2) {
        // page ids of every chunk of the wave, 16 lanes a chunk
#pragma unroll
        for (int c0 = 0; c0 < kChunks; c0 += 4) {
            const int c = c0 + kq, cr = (c % kPerTile) * G;
            const int first = __shfl(base, (cr >> 2) * 16 + (c / kPerTile) * 4 + (cr & 3), 64) >> rows.page_log2;
            // entries beyond the sequence's length are not read
            pages[c * kDecodePages + n] = rows.table[min(first + n, (pr.hi - 1) >> rows.page_log2)];
        }
        asm volatile("" ::: "memory");        // lanes read what other lanes of the wave wrote (LDS keeps the order)
    }
    // offset of row `pos` of this lane's chunk
    auto row_at = [&](int pos) -> off_t {
        if constexpr (SRC == 2) {
            const int idx = (pos >> rows.page_log2) - (base >> rows.page_log2);
            int page = pages[ci * kDecodePages + min(idx, kDecodePages - 1)];
            if (idx >= kDecodePages) page = rows.table[pos >> rows.page_log2];      // a chunk of more pages than that
            return rows.at(pos, page);
        } else if constexpr (SRC == 1) {
            return rows.at(pos, rows.src.slot_of(max(pos, 0)));
        } else {
            return rows.at(pos, 0);
        }
    };
    uint4 *staged = &sh_rows[wv * 16 * decode_row_pieces(KV8)];
    auto products = [&](uint4 (&raw)[kLoads]) {
        arrange_tile<KV8>(staged, n, kq, raw);
        return decode_products<KV8, PARTS>(raw, q);
    };
    // a tile's products -> the owners' scores (sL: against the column's query, or q_L; sR: against q_R).  i: the owner's
    // register; ix, i4: the registers that the owners in lanes n ^ 8 and n ^ 4 want
    auto owned = [&](const f32x4 c, int i, int ix, int i4, float &sL, float &sR) {
        auto of_head = [&](int r, int r4) {
            const float v = pick4(c, r);
            if constexpr (G < 8) return v;
            const float w = other_quad(pick4(c, r4));        // heads 0..3 are in the even quads' columns, and in rows of even kq
            return ((quad ^ kq) & 1) ? w : v;
        };
        const float v = of_head(i, i4);
        if constexpr (ROPE) {
            const float w = row_ror8(i == ix ? v : of_head(ix, i4 ^ i ^ ix));
            sL = n < 8 ? v : w;
            sR = n < 8 ? w : v;
        } else {
            sL = sR = v;
        }
    };
    // scores of the lanes' rows at `off`
    auto score = [&](off_t off, float &sL, float &sR) {
        uint4 raw[NT][kLoads];
        for_each_tile<NT>([&](auto t) { request_tile<t, KV8>(rows, off, n, raw[t]); });
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float l, rr;
            owned(products(raw[t]), n & 3, n & 3, n & 3, l, rr);
            sL = quad == t ? l : sL;
            sR = quad == t ? rr : sR;
        }
    };

    int half = a.chunk >> 1, off = 0;
    // left: the left key's score as a left branch; value: what the chunk score takes from this head
    float left = 0.f, value = 0.f, rL = 0.f, rR = 0.f;
    const bool has_right = half >= 1 && half < len;
    if constexpr (SRC == 1) {
        // both rows of a search on their way at once
        const int mid = has_right ? base + half : -1;
        const int slot0 = rows.src.slot_of(max(base, 0)), slot1 = rows.src.slot_of(max(mid, 0));
        uint4 r0[kLoads], r1[kLoads];
        request_tile<0, KV8>(rows, rows.at(base, slot0), n, r0);
        request_tile<0, KV8>(rows, rows.at(mid, slot1), n, r1);
        owned(products(r0), n & 3, n & 3, n & 3, left, value);
        owned(products(r1), n & 3, n & 3, n & 3, rL, rR);
    } else {
        const off_t at0 = row_at(base), at1 = row_at(has_right ? base + half : base);
        if constexpr (G >= 4) {
            // The first key of a chunk and of its right half are the same rows for all heads: one tile holds the first keys of the
            // wave's chunks, row 4*kq + t that of the chunk of quad t in row group kq (four heads: 16 chunks; eight: 8, each in
            // two row groups), so that the owner finds its score in register t.  Eight heads, a tile for each owner's first key / so (us),
            // 16 sequences of 8 KV heads, 8,192 chunks of two keys each: E4M3 175 / 108, bf16 pages with RoPE 350 / 218.
            auto first_of = [&](off_t at) {           // lane t of a row group: the offset of its lane 4 * t
                const off_t a0 = row_lane<0>(at), a1 = row_lane<4>(at), a2 = row_lane<8>(at), a3 = row_lane<12>(at);   // (by all lanes)
                return (n & 2) ? ((n & 1) ? a3 : a2) : (n & 1) ? a1 : a0;
            };
            uint4 r0[kLoads], r1[kLoads];
            request_tile<0, KV8>(rows, first_of(at0), n, r0);
            request_tile<0, KV8>(rows, first_of(at1), n, r1);
            owned(products(r0), quad, quad ^ 2, quad ^ 1, left, value);
            owned(products(r1), quad, quad ^ 2, quad ^ 1, rL, rR);
        } else {
            score(at0, left, value);
            score(at1, rL, rR);
        }
    }
    if (has_right && rR > left) { off = half; left = rL; value = rR; }        // strict: tie keeps left
    for (half >>= 1; half >= 1; half >>= 1) {
        const bool ok = off + half < len;
        score(row_at(ok ? start + off + half : unread), rL, rR);
        if (ok && rR > left) { off += half; left = rL; value = rR; }
    }

    if (a.out_rep != nullptr && owner && j < a.max_chunks) {
        const int64_t row = (int64_t)(pr.b * a.ge.Hq + pr.g * G + hd) * a.ge.Mq + pr.m;
        a.out_rep[row * a.max_chunks + j] = valid ? start + off : -1;
    }
    // chunk score: max over the heads
    float best = value;
    if constexpr (G >= 2) best = fmaxf(best, dpp_f32<0xB1>(best));
    if constexpr (G >= 4) best = fmaxf(best, dpp_f32<0x4E>(best));
    if constexpr (G == 8) best = fmaxf(best, __shfl_xor(best, 16, 64));
    if (owner && hd == 0 && j < a.max_chunks) a.out_scores[(int64_t)p * a.max_chunks + j] = valid ? (KV8 ? best * a.k_scale : best) : -INFINITY;
}

// Chunks of four keys: the search reads every row of a chunk anyway (all four unless the heads agree), so a tile is four
// whole chunks, and a head's four scores of a chunk are the four registers of one lane: no dependent loads.
template <int G, bool ROPE, int SRC, bool KV8, bool NARROW>
__global__ __launch_bounds__(256, !ROPE && !KV8 ? 5 : 1) void prune_decode_four_kernel(const PruneArgs a, const RopeView rope)
{
    static_assert(SRC == 0 || !NARROW, "paged pools are addressed with 64-bit offsets");
    constexpr int PARTS = ROPE ? 3 : 1;
    constexpr int NT = decode_tile_chunks(G, 4, ROPE, KV8) / 4;  // tiles of a wave, all in flight at once
    constexpr int kLoads = KV8 ? 2 : 4;
    using Rows = DecodeRows<SRC, NARROW>;
    const int p = a.grid.problem();
    const Problem pr = problem_of(a.ge, p);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const int j0 = (a.grid.part() * (blockDim.x >> 6) + wv) * NT * 4;
    if (j0 >= a.max_chunks) return;
    const Rows rows(a, pr);
    // Lane (n, kq) finds row 4 * kq + n % 4 of tile n / 4: key n % 4 of chunk kq of the tile (its first key where the chunk is cut
    // short; without a chunk key 0 of the sequence, unless the whole wave has none: see prune_decode_tile_kernel)
    const int j_own = j0 + (n >> 2) * 4 + kq;
    const int start_own = (n >> 2) < NT && j_own < a.max_chunks ? slot_start(pr, a.parent_starts, a.n_parent, a.ratio_log2, a.chunk, p, j_own) : -1;
    const int key = start_own >= 0 ? (start_own + (n & 3) < pr.hi ? start_own + (n & 3) : start_own) : 0;
    if (__ballot(start_own >= 0) == 0) {
        write_no_chunks<G>(a, pr, p, j0, NT * 4);
        return;
    }
    const int hd = G == 8 ? (n & 7) : n % G;
    bf16x8 q[PARTS][4];
    decode_query_operands<KV8, PARTS>(a.q + pr.b * a.q_sb + (int64_t)(pr.g * G + hd) * a.q_sh + (int64_t)pr.m * a.q_st, kq, rope,
                                      a.ge.n_stream + (n < 8 ? 1 : 0), q);
    __shared__ uint4 sh_rows[kDecodeTileWaves * 16 * decode_row_pieces(KV8)];
    uint4 *staged = &sh_rows[wv * 16 * decode_row_pieces(KV8)];
    uint4 raw[NT][kLoads];
    int page = 0;
    if constexpr (SRC == 2) page = rows.table[key >> rows.page_log2];
    const auto off_own = rows.at(key, page);
    for_each_tile<NT>([&](auto t) { request_tile<t, KV8>(rows, off_own, n, raw[t]); });
    int starts[NT];
    for_each_tile<NT>([&](auto t) { starts[t] = row_lane<4 * t>(start_own); });
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int j = j0 + t * 4 + kq, start = starts[t];       // as the owner: chunk kq of the tile, column n's head
        const int len = start >= 0 ? min(4, pr.hi - start) : 0;
        arrange_tile<KV8>(staged, n, kq, raw[t]);
        const f32x4 c = decode_products<KV8, PARTS>(raw[t], q);
        f32x4 sL = c, sR = c;
        if constexpr (ROPE) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float w = row_ror8(c[i]);
                sL[i] = n < 8 ? c[i] : w;
                sR[i] = n < 8 ? w : c[i];
            }
        }
        // the halving search over keys 0..3
        const bool right = 2 < len && sR[2] > sL[0];                          // strict: tie keeps left
        float left = right ? sL[2] : sL[0], best = right ? sR[2] : sR[0];
        int off = right ? 2 : 0;
        const float next = right ? sR[3] : sR[1];
        if (off + 1 < len && next > left) { off += 1; best = next; }
        if (a.out_rep != nullptr && j < a.max_chunks && n < G) {
            const int64_t row = (int64_t)(pr.b * a.ge.Hq + pr.g * G + hd) * a.ge.Mq + pr.m;
            a.out_rep[row * a.max_chunks + j] = start >= 0 ? start + off : -1;
        }
        if constexpr (G >= 2) best = fmaxf(best, dpp_f32<0xB1>(best));
        if constexpr (G >= 4) best = fmaxf(best, dpp_f32<0x4E>(best));
        if constexpr (G == 8) best = fmaxf(best, other_quad(best));
        if (n == 0 && j < a.max_chunks) a.out_scores[(int64_t)p * a.max_chunks + j] = start >= 0 ? (KV8 ? best * a.k_scale : best) : -INFINITY;
    }
}

// b_q == 1, K through strides or pages; SRC 1: behind the host tier, where chunks of four are searched too (only the rows that
// the search reads may be noted as touched)
template <int G, bool ROPE, int SRC, bool KV8, bool NARROW>
static void launch_decode_tile_n(PruneArgs a, const RopeView &rope, int P, hipStream_t st)
{
    const int per_wg = (SRC == 1 ? decode_search_tiles(SRC) * 16 / G : decode_tile_chunks(G, a.chunk, ROPE, KV8)) * kDecodeTileWaves;
    const int per_problem = (a.max_chunks + per_wg - 1) / per_wg;
    a.grid = prune_grid(a, P, per_problem, KV8, ROPE);
    const dim3 grid = a.grid.dims(P, per_problem), block(64 * kDecodeTileWaves);
    KernelTimer timer(stage_name(kNamePruneDecode, a.parent_starts == nullptr, a.chunk), st);
    if constexpr (SRC != 1) {
        if (a.chunk == 4) {
            hipLaunchKernelGGL((prune_decode_four_kernel<G, ROPE, SRC, KV8, NARROW>), grid, block, 0, st, a, rope);
            return;
        }
    }
    hipLaunchKernelGGL((prune_decode_tile_kernel<G, ROPE, SRC, KV8, NARROW>), grid, block, 0, st, a, rope);
}

template <bool ROPE, int SRC, bool KV8, bool NARROW>
static void launch_decode_tile_g(const PruneArgs &a, const RopeView &rope, int P, hipStream_t st)
{
    if constexpr (KV8) {                      // one and two heads: E4M3 rows only (decode_on_tiles)
        if (a.ge.G == 1) return launch_decode_tile_n<1, ROPE, SRC, KV8, NARROW>(a, rope, P, st);
        if (a.ge.G == 2) return launch_decode_tile_n<2, ROPE, SRC, KV8, NARROW>(a, rope, P, st);
    }
    if (a.ge.G == 4) launch_decode_tile_n<4, ROPE, SRC, KV8, NARROW>(a, rope, P, st);
    else launch_decode_tile_n<8, ROPE, SRC, KV8, NARROW>(a, rope, P, st);
}

template <bool ROPE, bool KV8>
static void launch_decode_tile_cached(const PruneArgs &a, const RopeView &rope, int P, hipStream_t st)
{
    switch (a.ge.G) {
    case 1: launch_decode_tile_n<1, ROPE, 1, KV8, false>(a, rope, P, st); break;
    case 2: launch_decode_tile_n<2, ROPE, 1, KV8, false>(a, rope, P, st); break;
    case 4: launch_decode_tile_n<4, ROPE, 1, KV8, false>(a, rope, P, st); break;
    default: launch_decode_tile_n<8, ROPE, 1, KV8, false>(a, rope, P, st); break;
    }
}

template <bool ROPE, bool KV8>
static void launch_decode_tile(const PruneArgs &a, const RopeView &rope, int P, int64_t max_seq_len, hipStream_t st)
{
    // byte offsets of 32 bits: every row of the slab within 4 GB of its base (strides are non-negative here or not narrow)
    const bool narrow = a.k_st >= 0 && max_seq_len * a.k_st * 2 + 512 < ((int64_t)1 << 32);
    if (a.paged.block_table != nullptr) launch_decode_tile_g<ROPE, 2, KV8, false>(a, rope, P, st);
    else if (narrow) launch_decode_tile_g<ROPE, 0, KV8, true>(a, rope, P, st);
    else launch_decode_tile_g<ROPE, 0, KV8, false>(a, rope, P, st);
}

}  // namespace ihip
