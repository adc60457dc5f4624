"""GPU parity of the chunked-prefill path with dynamic RoPE (Sec. 4 "Dynamic
RoPE for OOL generalization": relative-style positions in the pruning stages,
streaming-style positions in the block-sparse attention) against the CPU
oracle, through the C ABI.

Bit-exact bar: integer-valued Q/K/V with a quarter-turn rotary table (cos and
sin are 0 or +-1: rotated vectors stay small integers, exact in bf16 and in
the fp32 accumulators of the matrix cores).  Real tables on Gaussian inputs,
against the oracle as it stands (rotations and dot products in fp32): the
pruning kernels keep every rotated operand as a bf16 value plus a bf16 rest,
so their scores agree with the oracle's to a few 2^-18 of sum |q_i||k_i| and
every problem's kept list has recall >= 0.99 at every stage; the attention
rounds its rotated operands to bf16 (no decision hangs on them) and its
outputs agree within 2e-2.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from workloads import configs, gen  # noqa: E402


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build(force=False)
    return oracle


def small(Tq=256, prefix=2048, b_q=64, B=1, Hq=32, Hkv=8, n_stream=256, stages=((64, 8), (16, 16)), **kw):
    return configs.shrink(configs.CFG4, B=B, Hq=Hq, Hkv=Hkv, T=prefix + Tq, Tq=Tq, b_q=b_q,
                          n_stream=n_stream, stages=stages, **kw)


def gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune="relative", attn=True, want_rep=True):
    qd, kd, vd, sld = [t.cuda() for t in (q, k, v, sl)]
    style = {None: ihip.ROPE_NONE, "relative": ihip.ROPE_RELATIVE, "chunk": ihip.ROPE_CHUNK_INDEXED}[prune]
    rp = ihip.Rope(cos.cuda(), sin.cuda(), style, ihip.ROPE_STREAMING if attn else ihip.ROPE_NONE)
    L = ihip.Layer(qd, kd, sld, w.b_q, w.n_sink, w.n_stream)
    stages, parents, pchunk = [], None, 0
    for (l_c, keep) in w.stages:
        scores, rep = L.prune_stage(qd, kd, l_c, parents, pchunk, want_rep=want_rep, rope=rp if prune else None)
        kept = L.select_blocks(scores, l_c, keep, parents, pchunk)
        stages.append((scores, rep, kept))
        parents, pchunk = kept, l_c
    out, lse = L.sparse_attn_prefill(qd, kd, vd, parents, pchunk, want_lse=True, rope=rp if attn else None)
    fused = L.prefill_layer(qd, kd, vd, [s[0] for s in w.stages], [s[1] for s in w.stages], rope=rp)
    torch.cuda.synchronize()
    return stages, out, lse, fused


def compare(w, o, stages, out, lse, exact, problems=None, score_tol=None, max_off=0.05, stagewise=False):
    """stagewise (inexact mode): a stage after the first is compared with the oracle's stage run on the
    list the kernel kept in the stage before, and end to end only where those lists are the oracle's."""
    G, Mq = w.G, w.Mq
    worst, min_recall = 0.0, 1.0
    n_off = n_all = n_hit = n_want = 0
    N = len(w.stages)
    if problems is None:
        problems = [(b, g, m) for b in range(w.B) for g in range(w.Hkv) for m in range(Mq)]
    for (b, g, m) in problems:
        p = (b * w.Hkv + g) * Mq + m
        pr = o.prune(b, g, m, w.stages)
        gpu_kept = []
        for i, st in enumerate(pr.stages):
            scores, rep, kept = stages[i]
            n = len(st.starts)
            sc = scores[p].cpu().numpy()
            kp = kept[p].cpu().numpy()
            gpu_kept.append(kp[kp >= 0].astype(np.int64))
            if exact:
                assert np.array_equal(sc[:n], st.scores), (b, g, m, i)
                assert np.isneginf(sc[n:]).all(), (b, g, m, i)
                if rep is not None:
                    rp = rep[b, g * G:(g + 1) * G, m].cpu().numpy()
                    assert np.array_equal(rp[:, :n], st.reps), (b, g, m, i)
                    assert (rp[:, n:] == -1).all()
                ks = st.kept_starts
                assert np.array_equal(kp[:len(ks)], ks), (b, g, m, i)
                assert (kp[len(ks):] == -1).all()
            else:
                if i == 0:
                    # a search that turns the other way at a near-tie ends at another representative
                    # and another score: such chunks must be rare, all others agree to rounding
                    off = np.abs(sc[:n] - st.scores) > score_tol
                    assert off.mean() <= 2 * max_off, (b, g, m, off.mean())
                    n_off += int(off.sum())
                    n_all += n
                want = st.kept_starts
                same_input = all(np.array_equal(gpu_kept[j], pr.stages[j].kept_starts) for j in range(i))
                if stagewise and i > 0 and not same_input:
                    cached = gpu_kept[:i] + [np.zeros(0, np.int64)] * (N - i)
                    want = o.prune_due(b, g, m, w.stages, [j == i for j in range(N)], cached)[0][i]
                want = set(want.tolist())
                got = set(gpu_kept[i].tolist())
                assert len(got) == len(want)
                min_recall = min(min_recall, len(got & want) / max(1, len(want)))
                n_hit += len(got & want)
                n_want += len(want)
        if out is None:
            continue
        if exact:
            ref, ref_lse = o.attend(b, g, m, pr.block_starts, pr.block_lens)       # [G, b_q, d]
        else:
            # where a near-tie made the kernel keep another block than the oracle, the attention is
            # checked on the blocks the kernel kept
            kp = gpu_kept[-1]
            hi = o.ranges(b, m)[1]
            ref, ref_lse = o.attend(b, g, m, kp, np.minimum(w.stages[-1][0], hi - kp).astype(np.int32))
        got = out[b, g * G:(g + 1) * G, m * w.b_q:(m + 1) * w.b_q].float().cpu().numpy()
        worst = max(worst, np.abs(got - ref).max())
        if exact:
            np.testing.assert_allclose(lse[b, g * G:(g + 1) * G, m * w.b_q:(m + 1) * w.b_q].cpu().numpy(),
                                       ref_lse, rtol=2e-5, atol=2e-5)
    assert n_off <= max_off * max(n_all, 1), (n_off, n_all)
    return worst, (min_recall, n_hit / max(n_want, 1))


@pytest.mark.parametrize("w", [
    small(),                                              # Llama shape, 4 query blocks
    small(prefix=2048 + 37, B=2, Hq=8, Hkv=2),            # ragged middle, two sequences
    small(b_q=32, Tq=128, Hq=8, Hkv=2),
    small(b_q=16, Tq=64, Hq=4, Hkv=2, stages=((32, 8), (8, 16), (2, 40))),
    small(Hq=8, Hkv=8, Tq=128),                           # G = 1
    small(Hq=16, Hkv=2, Tq=64),                           # G = 8
    small(Hq=4, Hkv=2, Tq=128),                           # G = 2
], ids=["llama", "ragged-b2", "bq32", "bq16-3stage", "g1", "g8", "g2"])
@pytest.mark.parametrize("prune", ["relative", "chunk"])
def test_quarter_turn_table_bit_exact(ihip, orc, w, prune):
    # 64-query blocks with the relative style run two waves per head (every G here: 1, 2, 4 and 8 heads in
    # two passes), which exchange their maxima; 32- and 16-query blocks and the chunk-indexed style one
    q, k, v, sl, _ = configs.make_inputs(w, 0, kind="int")
    if w.B == 2:
        sl = torch.tensor([w.T, w.T - 517], dtype=torch.int32)
    cos, sin = gen.quarter_turn_table(w.T, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune=prune, attn="streaming"))
    stages, out, lse, fused = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune=prune)
    worst, _ = compare(w, o, stages, out, lse, exact=True)
    assert worst <= 2e-2
    assert torch.equal(fused, out)          # the one-enqueue layer call runs the same kernels


@pytest.mark.parametrize("fp8", [False, True])
def test_two_waves_per_head_give_the_same_result_every_time(ihip, fp8):
    """Relative style on 64-query blocks: the two waves of a head exchange their maxima by a handshake
    whose timing differs from run to run; scores and representatives must not.  A shape with many
    workgroups per CU, Gaussian values (no ties to hide a missed exchange), 12 runs of both stages."""
    w = small(Tq=1024, prefix=16384, stages=((64, 64), (16, 128)))
    q, k, v, sl, _ = configs.make_inputs(w, 4)
    cos, sin = gen.rope_table(4096, w.d)
    qd, sld = q.cuda(), sl.cuda()
    kd = gen.to_e4m3(k, 1.0 / 64).cuda() if fp8 else k.cuda()
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_NONE)
    L = ihip.Layer(qd, kd, sld, w.b_q, w.n_sink, w.n_stream)
    first = None
    for run in range(12):
        if fp8:
            blocks = torch.empty((L.P, w.stages[-1][1]), dtype=torch.int32, device="cuda")
            out = L.prefill_layer(qd, kd, kd, [s[0] for s in w.stages], [s[1] for s in w.stages], rope=rp,
                                  kv_scales=(1.0 / 64, 1.0 / 64), out_blocks=blocks)       # V = the same bytes
            cur = (out, blocks)
        else:
            scores, rep = L.prune_stage(qd, kd, 64, want_rep=True, rope=rp)
            kept = L.select_blocks(scores, 64, w.stages[0][1])
            scores2, rep2 = L.prune_stage(qd, kd, 16, kept, 64, want_rep=True, rope=rp)
            cur = (scores, rep, scores2, rep2)
        torch.cuda.synchronize()
        if first is None:
            first = [t.clone() for t in cur]
        else:
            for a, b in zip(first, cur):
                assert torch.equal(a, b), run


def test_rope_changes_selection_and_output(ihip, orc):
    # guards against a path that silently ignores the table
    w = small(Tq=128, prefix=2048)
    q, k, v, sl, _ = configs.make_inputs(w, 0, kind="int")
    cos, sin = gen.quarter_turn_table(w.T, w.d)
    with_rope = gpu_prefill(ihip, w, q, k, v, sl, cos, sin)
    without = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune=None, attn=False)
    assert not torch.equal(with_rope[0][0][0], without[0][0][0])
    assert not torch.equal(with_rope[1], without[1])


@pytest.mark.parametrize("prune", ["relative", "chunk"])
@pytest.mark.parametrize("seed", [0, 1])
def test_real_table_gaussian_recall_and_output(ihip, orc, seed, prune):
    # 256 / 257 first-stage chunks per problem of which 128 are kept, then 256 of 512: one chunk that
    # changes sides costs a problem less than 1 % of its recall.
    w = small(Tq=128, prefix=16384 + 320, Hq=16, Hkv=4, stages=((64, 128), (16, 256)))
    q, k, v, sl, _ = configs.make_inputs(w, seed)
    cos, sin = gen.rope_table(w.T, w.d)
    # The oracle as it stands: rotations and dot products in fp32.  A rotated operand of the kernels is
    # a bf16 value plus the bf16-rounded rest, i.e. within 2^-18 of its fp32 value, relatively; with
    # both sides and the dropped product of the two rests that bounds the difference of a score by
    # 3 * 2^-18 * sum |q_i||k_i| <= 3 * 2^-18 * |q||k| ~ 2e-3 for these vectors (|q|, |k| <= 13),
    # typically a tenth of that.  Chunks beyond it are those whose search turned the other way at
    # a near-tie and ended at another representative: at most 1 in 100.
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune=prune, attn="streaming"))
    stages, out, lse, fused = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune=prune, want_rep=False)
    # Chunk-indexed style: a key's position is the index of its chunk in the stage's list, so a single
    # chunk that changes sides at a near-tie of the stage before renumbers every chunk behind it and
    # the two runs score different problems from there on.  A later stage is therefore held against
    # the oracle's stage on the list the kernel kept before it (and end to end wherever the lists
    # agree); the relative style has no such coupling and is compared end to end throughout.
    worst, (min_recall, recall) = compare(w, o, stages, out, lse, exact=False, score_tol=2e-3, max_off=0.01,
                                          stagewise=prune == "chunk")
    assert min_recall >= 0.99           # every (sequence, KV head, query block) problem, every stage
    assert worst <= 2e-2


def test_streaming_attention_alone_on_oracle_indices(ihip, orc):
    # few kept blocks and many empty slots in the block list: window keys must skip them when numbered
    w = small(Tq=128, prefix=1500, Hq=8, Hkv=2, stages=((64, 6), (16, 40)))
    q, k, v, sl, _ = configs.make_inputs(w, 2)
    cos, sin = gen.rope_table(4096, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), attn="streaming"))
    qd, kd, vd, sld = [t.cuda() for t in (q, k, v, sl)]
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
    L = ihip.Layer(qd, kd, sld, w.b_q, w.n_sink, w.n_stream)
    n_slots = w.stages[-1][1]
    starts = np.full((w.Hkv * w.Mq, n_slots), -1, np.int32)
    refs = {}
    for g in range(w.Hkv):
        for m in range(w.Mq):
            pr = o.prune(0, g, m, w.stages)
            bs = pr.block_starts
            starts[g * w.Mq + m, :len(bs)] = bs
            refs[(g, m)] = o.attend(0, g, m, pr.block_starts, pr.block_lens)[0]
    assert (starts[:, -1] == -1).all()      # the case really has empty slots
    out, _ = L.sparse_attn_prefill(qd, kd, vd, torch.from_numpy(starts).cuda(), w.stages[-1][0], rope=rp)
    torch.cuda.synchronize()
    for (g, m), ref in refs.items():
        got = out[0, g * w.G:(g + 1) * w.G, m * w.b_q:(m + 1) * w.b_q].float().cpu().numpy()
        assert np.abs(got - ref).max() <= 2e-2


@pytest.mark.parametrize("variant", ["bf16", "fp8", "paged"])
@pytest.mark.parametrize("b_q,Hq,Hkv", [(64, 2, 2), (32, 2, 2), (32, 4, 2), (64, 4, 2)], ids=["bq64-g1", "bq32-g1", "bq32-g2", "bq64-g2"])
def test_streaming_attention_of_one_two_and_four_waves(ihip, orc, b_q, Hq, Hkv, variant):
    """The rotations of one- and two-wave workgroups take another loop body than those of four and more; several tiles, a
    masked and an unmasked one, first and last.  2e-2 as above: operands rounded to bf16 after their rotation."""
    w = small(Tq=128, prefix=1500, b_q=b_q, Hq=Hq, Hkv=Hkv, stages=((64, 6), (16, 20)))
    q, k, v, sl, _ = configs.make_inputs(w, 9)
    cos, sin = gen.rope_table(2048, w.d)
    scales = (1.0 / 32, 1.0 / 64) if variant == "fp8" else None
    if scales:
        k, v = gen.to_e4m3(k, scales[0]), gen.to_e4m3(v, scales[1])
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), attn="streaming"), kv_scales=scales)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    paged = None
    if variant == "paged":
        n = -(-w.T // 16)
        order = gen.distinct_ints(4, 5, n, n + 3)
        pools = []
        for t in (k, v):
            pool = torch.full((n + 3, w.Hkv, 16, w.d), 7.0, dtype=torch.bfloat16)
            pool[order] = torch.nn.functional.pad(t[0], (0, 0, 0, n * 16 - w.T)).view(w.Hkv, n, 16, w.d).permute(1, 0, 2, 3)
            pools.append(pool.cuda())
        paged = ihip.PagedKV(pools[0], pools[1], order.to(torch.int32).view(1, n).cuda())
    L = ihip.Layer(qd, kd, sl.cuda(), w.b_q, w.n_sink, w.n_stream)
    starts = np.full((w.Hkv * w.Mq, 20), -1, np.int32)
    refs = {}
    for g in range(w.Hkv):
        for m in range(w.Mq):
            pr = o.prune(0, g, m, w.stages)
            starts[g * w.Mq + m, :len(pr.block_starts)] = pr.block_starts
            refs[(g, m)] = o.attend(0, g, m, pr.block_starts, pr.block_lens)[0]
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
    out, _ = L.sparse_attn_prefill(qd, kd, vd, torch.from_numpy(starts).cuda(), 16, rope=rp, paged=paged, kv_scales=scales)
    torch.cuda.synchronize()
    for (g, m), ref in refs.items():
        got = out[0, g * w.G:(g + 1) * w.G, m * w.b_q:(m + 1) * w.b_q].float().cpu().numpy()
        assert np.abs(got - ref).max() <= 2e-2, (g, m)


def rotary(x, cos, sin, positions):
    """Standard RoPE in fp64: pair (2j, 2j+1) of row t turned by the table row of positions[t]."""
    c = cos[positions].double().view(1, 1, -1, cos.shape[1])
    s = sin[positions].double().view(1, 1, -1, sin.shape[1])
    xe, xo = x.double()[..., 0::2], x.double()[..., 1::2]
    out = torch.empty_like(x, dtype=torch.float64)
    out[..., 0::2] = xe * c - xo * s
    out[..., 1::2] = xe * s + xo * c
    return out


@pytest.mark.parametrize("prefix,prune", [(0, None), (0, "chunk"), (100, "relative"), (100, "chunk"), (1000, None),
                                          (1000, "chunk"), (19000, None), (23488, None), (23552, None)])
def test_keep_everything_with_streaming_ids_is_rotary_attention(ihip, prefix, prune):
    # When every chunk is kept a query attends to all keys before it, so the streaming ids are the
    # positions themselves and the result is ordinary causal attention on rotary-embedded q and k,
    # computed here by torch in fp64 without the oracle.
    # prefix 23488: 24,320 key slots, the most below what the 32x32 kernel keeps in LDS with RoPE (24,352);
    # prefix 23552: one chunk more -> the 16x16 kernel runs.  prefix 0 / 100: prefill from scratch, early
    # query blocks have an empty middle range and see only part of the sink.  With everything kept the
    # pruning style cannot change the result; it is varied to run those kernels on the edge shapes.
    keep = (prefix + 512) // 64 + 1
    w = small(Tq=512, prefix=prefix, n_stream=128, stages=((64, keep), (16, 4 * keep)))
    q, k, v, sl, _ = configs.make_inputs(w, 5)
    cos, sin = gen.rope_table(max(w.T, w.n_sink + 4 * keep * 16 + w.n_stream), w.d)     # a row per key slot
    qd, kd, vd, sld = [t.cuda() for t in (q, k, v, sl)]
    style = {None: ihip.ROPE_NONE, "relative": ihip.ROPE_RELATIVE, "chunk": ihip.ROPE_CHUNK_INDEXED}[prune]
    rp = ihip.Rope(cos.cuda(), sin.cuda(), style, ihip.ROPE_STREAMING)
    L = ihip.Layer(qd, kd, sld, w.b_q, w.n_sink, w.n_stream)
    out = L.prefill_layer(qd, kd, vd, [s[0] for s in w.stages], [s[1] for s in w.stages], rope=rp)
    torch.cuda.synchronize()
    G, T, Tq = w.G, w.T, w.Tq
    qr = rotary(q, cos, sin, torch.arange(T - Tq, T))
    kr = rotary(k, cos, sin, torch.arange(T))
    mask = torch.arange(T).view(1, -1) <= torch.arange(T - Tq, T).view(-1, 1)
    ref = torch.nn.functional.scaled_dot_product_attention(
        qr, kr.repeat_interleave(G, 1), v.double().repeat_interleave(G, 1), attn_mask=mask)
    assert (out.cpu().double() - ref).abs().max().item() <= 2e-2


@pytest.mark.parametrize("b_q,Hq,Hkv", [(64, 8, 2), (64, 16, 2), (32, 8, 2), (16, 4, 4)], ids=["bq64", "bq64-g8", "bq32", "bq16-g1"])
@pytest.mark.parametrize("stages", [((4, 8), (1, 16)), ((1, 40),)], ids=["4-1", "1"])
def test_chunk_indexed_queries_before_the_cap(ihip, orc, b_q, Hq, Hkv, stages):
    """A prompt from its first token, no sink, a window of one block: the second blocks' middle ranges hold so few
    keys that their first queries stand before n_chunk - 1 + n_stream (with one-key chunks every block's do) and
    keep their own positions, while later blocks share the capped one.  Exact on the quarter-turn table; on a real
    table first-stage scores within 3 * 2^-18 |q||k| (|q||k| <= 200 here)."""
    w = small(Tq=256, prefix=0, b_q=b_q, Hq=Hq, Hkv=Hkv, n_stream=64, n_sink=0, stages=stages)
    q, k, v, sl, _ = configs.make_inputs(w, 3, kind="int")
    cos, sin = gen.quarter_turn_table(w.T + 64, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune="chunk", attn="streaming"))
    st, out, lse, _ = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune="chunk")
    compare(w, o, st, out, lse, exact=True)
    q, k, v, sl, _ = configs.make_inputs(w, 4)
    cos, sin = gen.rope_table(w.T + 64, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune="chunk", attn="streaming"))
    st, _, _, _ = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune="chunk")
    _, (min_recall, _) = compare(w, o, st, None, None, exact=False, score_tol=2.3e-3, max_off=0.02, stagewise=True)
    assert min_recall >= 0.9


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (4, 2), (8, 2), (16, 2)], ids=["g1", "g2", "g4", "g8"])
@pytest.mark.parametrize("stages", [((4, 65), (2, 97), (1, 150)), ((2, 130),), ((1, 300),), ((8, 70), (4, 70)), ((256, 3), (32, 20))],
                         ids=["4-2-1", "2", "1", "8-4", "256-32"])
def test_relative_64_query_blocks_at_the_edges(ihip, orc, Hq, Hkv, stages):
    """The kernel of 64-query blocks, few workgroups (32 chunks per wave): chunks of one and two keys (no level after the
    first comparison picks up the late scores), slot counts around 64 and 128, a last chunk cut short, empty slots.
    Exact on the quarter-turn table."""
    relative_64_case(ihip, orc, small(Tq=192, prefix=701, Hq=Hq, Hkv=Hkv, n_stream=100, n_sink=33, stages=stages))


@pytest.mark.parametrize("kw", [
    dict(Hq=8, Hkv=8, B=2, prefix=701, stages=((1, 300),)),
    dict(Hq=4, Hkv=2, B=2, prefix=1701, stages=((2, 530), (1, 600))),
    dict(Hq=8, Hkv=2, B=2, prefix=3701, stages=((4, 430), (2, 450), (1, 500))),
    dict(Hq=16, Hkv=2, B=1, prefix=1701, stages=((1, 1700),)),
    dict(Hq=8, Hkv=2, B=1, Tq=1024, prefix=4701, stages=((16, 100), (4, 160))),
], ids=["g1-1", "g2-2-1", "g4-4-2-1", "g8-1", "g4-16-4"])
def test_relative_64_query_blocks_many_workgroups(ihip, orc, kw):
    """The same with more workgroups than run at once: 64 chunks per wave."""
    relative_64_case(ihip, orc, small(**{"Tq": 192, "n_stream": 100, "n_sink": 33, **kw}))


def relative_64_case(ihip, orc, w):
    q, k, v, sl, _ = configs.make_inputs(w, 6, kind="int")
    cos, sin = gen.quarter_turn_table(w.T + 128, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), w.b_q, w.n_sink, w.n_stream,
                   rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune="relative", attn="streaming"))
    st, out, lse, _ = gpu_prefill(ihip, w, q, k, v, sl, cos, sin, prune="relative")
    compare(w, o, st, out, lse, exact=True)
