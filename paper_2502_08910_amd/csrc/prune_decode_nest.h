// All stages of a decode plan in one pass over the middle range, or its last two in one over the chunks kept before them (b_q == 1, K from
// device memory, no RoPE or the relative style).
//
// SelectRep of a chunk compares the first keys of its halves and goes on inside the winner, so what it does inside a
// part is SelectRep of that part: once the parts of a chunk have their scores, the chunk's is that of one of them, chosen by the
// first keys alone.  A stage whose chunks are the parts of another stage's chunks can therefore be scored together with it,
// before the other's selection is known: every key is read once, in order, and all levels follow from the
// keys' scores in the registers.  Keys of parts that the selections drop are read for nothing; what it saves is a chain:
// log2(l) row latencies per stage become one, and all launches but one and all selections' but one (select_chain.hip) go.
// Layers of three stages, 32 heads on 8, stage by stage / in one pass (us): one sequence of 5K bf16 keys 35.1 / 22.7, 10K
// 36.5 / 24.3, 39K 39.0 / 35.7, 10 of 4K 57.4 / 39.1, 14 of 8K 96.6 / 69.9.
// The last two stages of longer plans (together_from in api.hip), 128 chunks of 64 kept, 256 of 16, 512 of 4: 13 sequences of 135K, E4M3
// pages 153.8 / 143.5; 256 of 64, 512 of 16, 1,024 of 4: 64 heads on 8, 5 of 835K, E4M3 pages 389 / 375, 8 of 1M bf16 437.6 / 433.4.
//
// Arithmetic as in prune_decode_tile.h: 16 keys x 16 query columns on the matrix cores; column n is head n % G (relative style:
// columns 0..7 against q_L, 8..15 against q_R, exchanged by a row rotation), and the lane (n, kq) holds keys 4*kq..+3
// of the tile: the last two levels of the search are in one lane, the levels of 8 and 16 keys compare kq with its
// partners (two row swaps), those of 32 and 64 a wave's four tiles, those of 128 and 256 the workgroup's four waves, through LDS.
#pragma once

#include "prune_decode_tile.h"
#include "prune_nest_args.h"

namespace ihip {

struct NestPart {
    float first_l, first_r, value;        // the first key as left and right branch; the part's score for this column's head
    int at;                               // position of the first key, -1 without one
};
template <bool ROPE>
__device__ inline NestPart nest_join(const NestPart &a, const NestPart &b)      // two halves, a the left one
{
    const bool right = b.at >= 0 && (ROPE ? b.first_r : b.first_l) > a.first_l;     // strict: tie keeps left
    return NestPart{a.first_l, a.first_r, right ? b.value : a.value, a.at};
}
// the halves in the rows kq and kq ^ 1 (D = 16) or kq ^ 2 (D = 32): every lane gets both, the left one first
template <int D>
__device__ inline void nest_swap(uint32_t v, uint32_t &l, uint32_t &r)
{
    if constexpr (D == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        l = s[0]; r = s[1];
    } else {
        const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        l = s[0]; r = s[1];
    }
}
template <int D, bool ROPE>
__device__ inline NestPart nest_join_rows(const NestPart &p)
{
    NestPart a, b;
    uint32_t l, r;
    nest_swap<D>(__float_as_uint(p.first_l), l, r);
    a.first_l = __uint_as_float(l); b.first_l = __uint_as_float(r);
    nest_swap<D>(__float_as_uint(p.value), l, r);
    a.value = __uint_as_float(l); b.value = __uint_as_float(r);
    nest_swap<D>((uint32_t)p.at, l, r);
    a.at = (int)l; b.at = (int)r;
    a.first_r = b.first_r = 0.f;
    if constexpr (ROPE) {
        nest_swap<D>(__float_as_uint(p.first_r), l, r);
        a.first_r = __uint_as_float(l); b.first_r = __uint_as_float(r);
    }
    return nest_join<ROPE>(a, b);
}

// PARENTS: the keys are those of the chunks that the stage before kept (as a branch of one kernel: passes over the middle range 1-2 % longer)
template <int G, bool ROPE, int SRC, bool KV8, bool NARROW, bool PARENTS>
__global__ __launch_bounds__(256) void prune_decode_nest_kernel(const PruneArgs a, const NestArgs nest, const RopeView rope)
{
    static_assert(SRC == 0 || !NARROW, "paged pools are addressed with 64-bit offsets");
    constexpr int PARTS = ROPE ? 3 : 1;
    constexpr int NT = 4;                     // 16-key tiles of a wave, all in flight at once
    constexpr int kLoads = KV8 ? 2 : 4;
    using Rows = DecodeRows<SRC, NARROW>;
    const int p = a.grid.problem();
    const Problem pr = problem_of(a.ge, p);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 15, kq = lane >> 4;
    const int log2l = nest.top + 2;
    // key f of the middle range, or of the parents one after the other, is key f % l of chunk f / l
    const int f0 = (a.grid.part() * 4 + wv) * (NT * 16), n_keys = a.max_chunks << log2l;
    const bool across = nest.top >= 5;        // the waves of the workgroup meet at the end
    if (f0 >= n_keys && !across) return;
    __shared__ float sh_part[4][4][16];
    __shared__ uint4 sh_rows[4 * 16 * decode_row_pieces(KV8)];
    // where the wave's keys begin: in the middle range, or inside one parent (of 64 keys or more)
    int w0 = pr.lo + f0;
    if constexpr (PARENTS) {
        const int parent_log2 = log2l + a.ratio_log2, i = f0 >> parent_log2;
        const int ps = i < a.n_parent ? a.parent_starts[(int64_t)p * a.n_parent + i] : -1;
        w0 = ps >= 0 ? ps + (f0 & ((1 << parent_log2) - 1)) : INT32_MAX - (NT * 16 - 1);     // no key of any sequence
    }
    auto position = [&](int f) { return f < n_keys && w0 + (f - f0) < pr.hi ? w0 + (f - f0) : -1; };
    NestPart whole{-INFINITY, -INFINITY, -INFINITY, -1};      // of the wave's 64 keys
    // chunk score of a part: max over the heads
    auto over_heads = [&](const NestPart &x) {
        float best = x.value;
        if constexpr (G >= 2) best = fmaxf(best, dpp_f32<0xB1>(best));
        if constexpr (G >= 4) best = fmaxf(best, dpp_f32<0x4E>(best));
        if constexpr (G == 8) best = fmaxf(best, other_quad(best));
        return x.at >= 0 ? (KV8 ? best * a.k_scale : best) : -INFINITY;
    };
    auto store = [&](int lv, bool mine, int j, float v) {
        if (mine && j < nest.slots[lv]) nest.out[lv][(int64_t)p * nest.stride + j] = v;
    };
    if (position(f0) < 0) {                   // no key at all: nothing may be read (see prune_decode_tile_kernel)
        const bool there = f0 < n_keys;
        if (nest.out[0]) store(0, there && lane < 16, (f0 >> 2) + lane, -INFINITY);
        if (nest.out[1]) store(1, there && lane < 8, (f0 >> 3) + lane, -INFINITY);
        if (nest.out[2]) store(2, there && lane < 4, (f0 >> 4) + lane, -INFINITY);
        if (nest.out[3]) store(3, there && lane < 2, (f0 >> 5) + lane, -INFINITY);
        if (nest.out[4]) store(4, there && lane < 1, f0 >> 6, -INFINITY);
    } else {
    const Rows rows(a, pr);
    uint4 raw[NT][kLoads];
    {
        // lane (n, kq) finds row 4 * kq + n % 4 of tile n / 4; without a key: key 0 of the sequence, which is there
        const int key = max(position(f0 + (n >> 2) * 16 + kq * 4 + (n & 3)), 0);
        int page = 0;
        if constexpr (SRC == 2) page = rows.table[key >> rows.page_log2];
        const auto off = rows.at(key, page);
        for_each_tile<NT>([&](auto t) { request_tile<t, KV8>(rows, off, n, raw[t]); });
    }
    uint4 *staged = &sh_rows[wv * 16 * decode_row_pieces(KV8)];
    const int hd = G == 8 ? (n & 7) : n % G;
    bf16x8 q[PARTS][4];
    decode_query_operands<KV8, PARTS>(a.q + pr.b * a.q_sb + (int64_t)(pr.g * G + hd) * a.q_sh + (int64_t)pr.m * a.q_st, kq, rope,
                                      a.ge.n_stream + (n < 8 ? 1 : 0), q);
    NestPart t0, t1, t2, t3;                  // of the tiles
    float s4[NT], s8[NT], s16[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
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
        const int first = position(f0 + t * 16 + 4 * kq);                    // position of this lane's first key
        const int len = first >= 0 ? min(4, pr.hi - first) : 0;
        const bool right = 2 < len && sR[2] > sL[0];                         // strict: tie keeps left
        const float left = right ? sL[2] : sL[0], next = right ? sR[3] : sR[1];
        const bool odd = (right ? 3 : 1) < len && next > left;
        NestPart x{sL[0], sR[0], odd ? next : right ? sR[2] : sR[0], first};
        s4[t] = over_heads(x);
        x = nest_join_rows<16, ROPE>(x);
        s8[t] = over_heads(x);
        x = nest_join_rows<32, ROPE>(x);
        s16[t] = over_heads(x);
        if (t == 0) t0 = x;
        else if (t == 1) t1 = x;
        else if (t == 2) t2 = x;
        else t3 = x;
    }
    if (nest.out[0]) store(0, n < NT, (f0 >> 2) + n * 4 + kq, n == 0 ? s4[0] : n == 1 ? s4[1] : n == 2 ? s4[2] : s4[3]);
    if (nest.out[1]) store(1, n < NT && (kq & 1) == 0, (f0 >> 3) + n * 2 + (kq >> 1), n == 0 ? s8[0] : n == 1 ? s8[1] : n == 2 ? s8[2] : s8[3]);
    if (nest.out[2]) store(2, n < NT && kq == 0, (f0 >> 4) + n, n == 0 ? s16[0] : n == 1 ? s16[1] : n == 2 ? s16[2] : s16[3]);
    if (nest.top >= 3) {
        const NestPart h0 = nest_join<ROPE>(t0, t1), h1 = nest_join<ROPE>(t2, t3);
        whole = nest_join<ROPE>(h0, h1);
        const float s0 = over_heads(h0), s1 = over_heads(h1), s64 = over_heads(whole);
        if (nest.out[3]) store(3, lane < 2, (f0 >> 5) + lane, lane == 0 ? s0 : s1);
        if (nest.out[4]) store(4, lane == 0, f0 >> 6, s64);
    }
    }
    if (!across) return;
    if (lane < 16) {
        sh_part[wv][0][lane] = whole.first_l;
        sh_part[wv][1][lane] = whole.first_r;
        sh_part[wv][2][lane] = whole.value;
        sh_part[wv][3][lane] = __int_as_float(whole.at);
    }
    __syncthreads();
    if (wv != 0) return;
    auto of_wave = [&](int w) { return NestPart{sh_part[w][0][n], sh_part[w][1][n], sh_part[w][2][n], __float_as_int(sh_part[w][3][n])}; };
    const NestPart h0 = nest_join<ROPE>(of_wave(0), of_wave(1)), h1 = nest_join<ROPE>(of_wave(2), of_wave(3));
    const float s0 = over_heads(h0), s1 = over_heads(h1), s256 = over_heads(nest_join<ROPE>(h0, h1));
    if (nest.out[5]) store(5, lane < 2, (f0 >> 7) + lane, lane == 0 ? s0 : s1);
    if (nest.out[6]) store(6, lane == 0, f0 >> 8, s256);
}

template <int G, bool ROPE, int SRC, bool KV8, bool NARROW>
static void launch_nest_n(PruneArgs a, const NestArgs &nest, const RopeView &rope, int P, hipStream_t st)
{
    const int per_problem = (int)((((int64_t)a.max_chunks << (nest.top + 2)) + 255) / 256);
    a.grid = DecodeGrid{0};                   // in order: a problem's keys by one XCD are 16 sequences of 16K keys 148 -> 178 us a layer
    KernelTimer timer(stage_name(kNamePruneDecode, a.parent_starts == nullptr, a.chunk), st);
    const dim3 grid = a.grid.dims(P, per_problem);
    if (a.parent_starts != nullptr) hipLaunchKernelGGL((prune_decode_nest_kernel<G, ROPE, SRC, KV8, NARROW, true>), grid, dim3(256), 0, st, a, nest, rope);
    else hipLaunchKernelGGL((prune_decode_nest_kernel<G, ROPE, SRC, KV8, NARROW, false>), grid, dim3(256), 0, st, a, nest, rope);
}
template <bool ROPE, int SRC, bool KV8, bool NARROW>
static void launch_nest_g(const PruneArgs &a, const NestArgs &nest, const RopeView &rope, int P, hipStream_t st)
{
    switch (a.ge.G) {
    case 1: launch_nest_n<1, ROPE, SRC, KV8, NARROW>(a, nest, rope, P, st); break;
    case 2: launch_nest_n<2, ROPE, SRC, KV8, NARROW>(a, nest, rope, P, st); break;
    case 4: launch_nest_n<4, ROPE, SRC, KV8, NARROW>(a, nest, rope, P, st); break;
    default: launch_nest_n<8, ROPE, SRC, KV8, NARROW>(a, nest, rope, P, st); break;
    }
}
template <bool ROPE, bool KV8>
static void launch_nest(const PruneArgs &a, const NestArgs &nest, const RopeView &rope, int P, int64_t max_seq_len, hipStream_t st)
{
    const bool narrow = a.k_st >= 0 && max_seq_len * a.k_st * 2 + 512 < ((int64_t)1 << 32);      // as in launch_decode_tile
    if (a.paged.block_table != nullptr) launch_nest_g<ROPE, 2, KV8, false>(a, nest, rope, P, st);
    else if (narrow) launch_nest_g<ROPE, 0, KV8, true>(a, nest, rope, P, st);
    else launch_nest_g<ROPE, 0, KV8, false>(a, nest, rope, P, st);
}

}  // namespace ihip
