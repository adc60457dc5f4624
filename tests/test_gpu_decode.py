"""GPU parity of the decode path against the CPU oracle, through the C ABI.

Bar: selected index sets, representatives and scores bit-exact on
integer-valued inputs (fp32 dot products are exact in any order); on Gaussian
inputs block recall >= 0.99 per problem and outputs within 2e-2 max-abs.
"""
import ctypes
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from workloads import configs, gen  # noqa: E402


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(scope="module")
def ihip():
    _need_gpu()
    import paper_2502_08910_amd as pkg
    pkg.lib()                       # raises if the HIP library is not built
    return pkg


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build(force=False)
    return oracle


def gpu_stagewise(ihip, w, q, k, v, seq_lens, want_rep=True):
    """Runs stage by stage through the separate entry points."""
    L = ihip.Layer(q, k, seq_lens, w.b_q, w.n_sink, w.n_stream)
    stages, parents, pchunk = [], None, 0
    for (l_c, keep) in w.stages:
        scores, rep = L.prune_stage(q, k, l_c, parents, pchunk, want_rep=want_rep)
        kept = L.select_blocks(scores, l_c, keep, parents, pchunk)
        stages.append((scores, rep, kept))
        parents, pchunk = kept, l_c
    out, lse = L.sparse_attn_decode(q, k, v, parents, pchunk, want_lse=True)
    torch.cuda.synchronize()
    return L, stages, out, lse


def compare_stagewise(w, o, stages, out, lse, exact, problems=None):
    """Element-by-element comparison with the oracle, problem by problem."""
    G = w.G
    worst, min_recall = 0.0, 1.0
    if problems is None:
        problems = [(b, g) for b in range(w.B) for g in range(w.Hkv)]
    for (b, g) in problems:
        p = b * w.Hkv + g
        pr = o.prune(b, g, 0, w.stages)
        for i, st in enumerate(pr.stages):
            scores, rep, kept = stages[i]
            n = len(st.starts)
            sc = scores[p].cpu().numpy()
            kp = kept[p].cpu().numpy()
            if exact:
                assert np.array_equal(sc[:n], st.scores), (b, g, i)
                assert np.isneginf(sc[n:]).all()
                if rep is not None:
                    rp = rep[b, g * G:(g + 1) * G, 0].cpu().numpy()
                    assert np.array_equal(rp[:, :n], st.reps), (b, g, i)
                    assert (rp[:, n:] == -1).all()
                ks = st.kept_starts
                assert np.array_equal(kp[:len(ks)], ks), (b, g, i)
                assert (kp[len(ks):] == -1).all()
            else:
                np.testing.assert_allclose(sc[:n], st.scores, rtol=1e-5, atol=1e-4)
                want = set(st.kept_starts.tolist())
                got = set(kp[kp >= 0].tolist())
                assert len(got) == len(want)
                min_recall = min(min_recall, len(got & want) / max(1, len(want)))
                assert (np.diff(kp[kp >= 0]) > 0).all()
        # attention over the oracle's own final blocks
        ref, ref_lse = o.attend(b, g, 0, pr.block_starts, pr.block_lens)
        got = out[b, g * G:(g + 1) * G, 0].float().cpu().numpy()
        worst = max(worst, np.abs(got - ref[:, 0]).max())
        if exact:
            np.testing.assert_allclose(lse[b, g * G:(g + 1) * G, 0].cpu().numpy(), ref_lse[:, 0],
                                       rtol=1e-5, atol=1e-5)
    return worst, min_recall


def dev(*ts):
    return [t.cuda() for t in ts]


# ---------------------------------------------------------------------------
@pytest.mark.parametrize("T,B", [(8192, 1), (8192 + 37, 2), (1500, 1)])
def test_integer_inputs_bit_exact(ihip, orc, T, B):
    w = configs.shrink(configs.CFG1, T=T, B=B, n_needles=0)
    q, k, v, sl, _ = configs.make_inputs(w, 0, kind="int")
    if B == 2:
        sl = torch.tensor([T, T - 1001], dtype=torch.int32)
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream)
    L, stages, out, lse = gpu_stagewise(ihip, w, *dev(q, k, v, sl))
    worst, _ = compare_stagewise(w, o, stages, out, lse, exact=True)
    assert worst <= 2e-2


@pytest.mark.parametrize("seed", [0, 1])
def test_gaussian_cfg1_recall_and_output(ihip, orc, seed):
    w = configs.CFG1
    q, k, v, sl, pos = configs.make_inputs(w, seed)
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream)
    L, stages, out, lse = gpu_stagewise(ihip, w, *dev(q, k, v, sl))
    # attention checked in isolation on the oracle's indices as well
    worst, recall = compare_stagewise(w, o, stages, out, lse, exact=False)
    assert recall >= 0.99
    assert worst <= 2e-2
    # needles survive on the GPU too
    final = stages[-1][2].cpu().numpy()
    l_n = w.stages[-1][0]
    for g in range(w.Hkv):
        kept = set((final[g][:, None] + np.arange(l_n)[None]).ravel().tolist())
        assert all(int(x) in kept for x in pos[0, g])


def test_attention_alone_on_oracle_indices(ihip, orc):
    w = configs.CFG1
    q, k, v, sl, _ = configs.make_inputs(w, 3)
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream)
    starts = np.full((w.Hkv, w.stages[-1][1]), -1, np.int32)
    refs = []
    for g in range(w.Hkv):
        pr = o.prune(0, g, 0, w.stages)
        starts[g, :len(pr.block_starts)] = pr.block_starts
        refs.append(o.attend(0, g, 0, pr.block_starts, pr.block_lens))
    qd, kd, vd, sld = dev(q, k, v, sl)
    L = ihip.Layer(qd, kd, sld, 1, w.n_sink, w.n_stream)
    out, lse = L.sparse_attn_decode(qd, kd, vd, torch.from_numpy(starts).cuda(), w.stages[-1][0], want_lse=True)
    for g in range(w.Hkv):
        got = out[0, g * w.G:(g + 1) * w.G, 0].float().cpu().numpy()
        assert np.abs(got - refs[g][0][:, 0]).max() <= 4e-3
        np.testing.assert_allclose(lse[0, g * w.G:(g + 1) * w.G, 0].cpu().numpy(), refs[g][1][:, 0],
                                   rtol=2e-5, atol=2e-5)


@pytest.mark.parametrize("T", [1, 5, 128, 129, 700, 1152, 1153, 1300])
def test_short_sequences(ihip, orc, T):
    # shorter than the sink, inside the window, a middle range of one ragged chunk, ...
    w = configs.shrink(configs.CFG1, T=max(T, 8), n_needles=0, stages=((64, 4), (16, 8), (4, 16)))
    q, k, v, _, _ = configs.make_inputs(w, 2, kind="int")
    sl = torch.tensor([T], dtype=torch.int32)
    o = orc.Oracle(q, k, v, [T], 1, w.n_sink, w.n_stream)
    L, stages, out, lse = gpu_stagewise(ihip, w, *dev(q, k, v, sl))
    worst, _ = compare_stagewise(w, o, stages, out, lse, exact=True)
    assert worst <= 2e-2


def test_keep_everything_is_dense(ihip, orc):
    w = configs.shrink(configs.CFG1, T=2048 + 5, n_stream=256, n_needles=0,
                       stages=((64, 1000), (16, 4000), (4, 16000)))
    q, k, v, sl, _ = configs.make_inputs(w, 5)
    qd, kd, vd, sld = dev(q, k, v, sl)
    L, stages, out, lse = gpu_stagewise(ihip, w, qd, kd, vd, sld, want_rep=False)
    G = w.G
    ref = torch.nn.functional.scaled_dot_product_attention(
        q.double(), k.double().repeat_interleave(G, 1), v.double().repeat_interleave(G, 1))
    assert (out.cpu().double() - ref).abs().max().item() <= 2e-2


def test_fused_entry_points_equal_stagewise(ihip, orc):
    w = configs.shrink(configs.CFG1, B=2, T=4096 + 11)
    q, k, v, sl, _ = configs.make_inputs(w, 4)
    sl = torch.tensor([w.T, w.T - 333], dtype=torch.int32)
    qd, kd, vd, sld = dev(q, k, v, sl)
    L, stages, out, lse = gpu_stagewise(ihip, w, qd, kd, vd, sld, want_rep=False)
    chunks = [s[0] for s in w.stages]
    keeps = [s[1] for s in w.stages]
    blocks = L.prune_all(qd, kd, chunks, keeps)
    assert torch.equal(blocks, stages[-1][2])
    blocks2 = torch.empty_like(blocks)
    out2 = L.decode_layer(qd, kd, vd, chunks, keeps, out_blocks=blocks2)
    torch.cuda.synchronize()
    assert torch.equal(blocks2, blocks)
    assert torch.equal(out2, out)
    # twice the same: deterministic
    out3 = L.decode_layer(qd, kd, vd, chunks, keeps)
    assert torch.equal(out3, out)


def test_strided_kv_layout(ihip, orc):
    # token-major storage [B,T,Hkv,d] viewed as [B,Hkv,T,d]
    w = configs.shrink(configs.CFG1, T=2048, n_stream=256, n_needles=0, stages=((64, 8), (16, 8), (4, 16)))
    q, k, v, sl, _ = configs.make_inputs(w, 6, kind="int")
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream)
    kd = k.cuda().permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    vd = v.cuda().permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert not kd.is_contiguous()
    L, stages, out, lse = gpu_stagewise(ihip, w, q.cuda(), kd, vd, sl.cuda())
    worst, _ = compare_stagewise(w, o, stages, out, lse, exact=True)
    assert worst <= 2e-2


def select_case(ihip, orc, P, n, keep, ties):
    rng = np.random.default_rng(n + keep + P)
    chunk, n_sink, n_stream = 4, 8, 16
    s = rng.standard_normal((P, n)).astype(np.float32)
    if ties:
        s = np.round(s * 2) / 2
        s[:, ::7] = -0.0
        s[:, 3::7] = 0.0
    n_valid = [(n, max(1, n - 5), max(1, n // 2))[p % 3] for p in range(P)]
    T = n_sink + n * chunk + n_stream
    seq = []
    for p in range(P):
        s[p, n_valid[p]:] = -np.inf
        seq.append(n_sink + n_valid[p] * chunk - (1 if n_valid[p] > 1 else 0) + n_stream)   # last chunk ragged
    q = torch.zeros((P, 1, 1, 128), dtype=torch.bfloat16).cuda()
    k = torch.zeros((1, 1, T, 128), dtype=torch.bfloat16).cuda().expand(P, 1, T, 128)      # never read
    L = ihip.Layer(q, k, torch.tensor(seq, dtype=torch.int32).cuda(), 1, n_sink, n_stream)
    got = L.select_blocks(torch.from_numpy(s).cuda(), chunk, keep).cpu().numpy()
    lib = orc.lib()
    for p in range(P):
        ids = np.empty(max(1, min(keep, n)), np.int32)
        cnt = lib.orc_topk(n_valid[p], s[p].ctypes.data_as(ctypes.c_void_p), keep,
                           ids.ctypes.data_as(ctypes.c_void_p))
        want = n_sink + ids[:cnt].astype(np.int64) * chunk
        assert np.array_equal(got[p, :cnt], want), p
        assert (got[p, cnt:] == -1).all()


@pytest.mark.parametrize("n,keep,ties", [(1, 1, False), (110, 64, False), (257, 64, True), (1000, 1000, True),
                                         (50, 80, True), (1500, 300, False), (2048, 512, True),
                                         (4092, 256, False), (4092, 256, True),
                                         (4143, 256, False), (6000, 2500, True), (8192, 300, True),
                                         (12288, 300, True), (20000, 777, True), (300, 1, True)])
def test_select_blocks_alone(ihip, orc, n, keep, ties):
    """Three problems: every workgroup shape of the selection that few problems get (4 slots per thread in
    256, 512 or 1024 threads, then 8 and 16 in 1024), the radix fallback beyond, heavy ties."""
    select_case(ihip, orc, 3, n, keep, ties)


@pytest.mark.parametrize("n,keep,ties", [(900, 100, False), (1500, 300, True), (3000, 256, False), (6000, 700, True),
                                         (12000, 300, False), (20000, 500, True)])
def test_select_blocks_many_problems(ihip, orc, n, keep, ties):
    """More problems than CUs: the smallest workgroup that holds the slots (256 threads with 4, 8 or 16
    slots each, 512 and 1024 threads with 16), and the radix select beyond."""
    select_case(ihip, orc, 260, n, keep, ties)


@pytest.mark.parametrize("n", [1025, 1536, 1537, 2049, 2560, 2561, 3073, 3584, 3585, 4096, 4097, 5120, 5121, 6145, 7168,
                               7169, 8193])
def test_select_blocks_slots_per_thread(ihip, orc, n):
    """Many problems: the edges between 6, 8, 10, 12, 14 and 16 slots per thread in 256 and 512 threads."""
    select_case(ihip, orc, 257, n, n // 7, n % 2 == 0)


def test_decode_layer_under_graph_capture(ihip, orc):
    """The fused layer call allocates nothing and never synchronises, so it can be captured into a
    HIP graph; every replay (with eager work in between, new queries written in place) must give
    the eager result."""
    w = configs.shrink(configs.CFG1, B=2, T=4096 + 7)
    chunks = [s[0] for s in w.stages]
    keeps = [s[1] for s in w.stages]
    q, k, v, sl, _ = configs.make_inputs(w, 7)
    qd, kd, vd, sld = dev(q, k, v, sl)
    L = ihip.Layer(qd, kd, sld, 1, w.n_sink, w.n_stream)
    ws = L.workspace(ihip.OP_DECODE_LAYER, chunks, keeps)
    out = torch.empty((w.B, w.Hq, 1, w.d), dtype=torch.bfloat16, device="cuda")
    blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                      # warm-up outside capture
        L.decode_layer(qd, kd, vd, chunks, keeps, ws=ws, out=out, out_blocks=blocks)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        L.decode_layer(qd, kd, vd, chunks, keeps, ws=ws, out=out, out_blocks=blocks)
    for seed in (11, 12, 13):
        qn = configs.make_q(w, seed).cuda()
        ref_blocks = torch.empty_like(blocks)
        ref = L.decode_layer(qn, kd, vd, chunks, keeps, out_blocks=ref_blocks)     # eager, own buffers
        qd.copy_(qn)                                    # new input written in place
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(blocks, ref_blocks), seed
        assert torch.equal(out, ref), seed


def test_empty_batch_is_a_no_op(ihip):
    # B = 0: every entry point returns without enqueuing anything or touching a pointer
    w = configs.shrink(configs.CFG1, T=2048, n_needles=0)
    q = torch.empty((0, w.Hq, 1, w.d), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((0, w.Hkv, w.T, w.d), dtype=torch.bfloat16, device="cuda")
    sl = torch.empty((0,), dtype=torch.int32, device="cuda")
    L = ihip.Layer(q, k, sl, 1, w.n_sink, w.n_stream)
    chunks, keeps = [s[0] for s in w.stages], [s[1] for s in w.stages]
    scores, _ = L.prune_stage(q, k, chunks[0])
    assert scores.shape[0] == 0
    kept = L.select_blocks(scores, chunks[0], keeps[0])
    assert kept.shape == (0, keeps[0])
    out = L.decode_layer(q, k, k, chunks, keeps)
    assert out.shape == (0, w.Hq, 1, w.d)
    Lp = ihip.Layer(torch.empty((0, w.Hq, 64, w.d), dtype=torch.bfloat16, device="cuda"), k, sl, 64, w.n_sink, 1024)
    outp = Lp.prefill_layer(torch.empty((0, w.Hq, 64, w.d), dtype=torch.bfloat16, device="cuda"), k, k, chunks, keeps)
    torch.cuda.synchronize()
    assert outp.shape == (0, w.Hq, 64, w.d)


@pytest.mark.parametrize("Hkv,G,n_blocks,block,n_stream", [
    (1, 4, 1024, 4, 1024),        # one problem: 55 splits of 96 slots
    (1, 8, 37, 16, 333),          # 17 splits, the last one of 13 slots: just past the one-group merge
    (8, 4, 128, 4, 1024),         # 26 splits
    (2, 1, 0, 4, 40),             # splits of 64 slots, no blocks
    (8, 2, 512, 8, 1000),         # the most splits
    (16, 2, 128, 8, 3200),        # 18 coarse splits each already fill the chip: the same splits either way
    (32, 1, 96, 4, 1152),         # 15 splits of 112 slots: two workgroups per compute unit, not more
], ids=["55", "17", "26", "short", "8x5k", "16x4k", "32x1.7k"])
def test_attention_splits_fine_and_coarse(ihip, orc, Hkv, G, n_blocks, block, n_stream):
    """The split of the key list follows the scratch: with what ihip_workspace_bytes says splits of 64 slots and more,
    with a byte less (and room for the coarse ones) of 256 and more, both against the oracle (4e-3, as every attention on
    given blocks here) and each other; less than the coarse ones need is refused."""
    w = configs.shrink(configs.CFG1, T=9001, Hq=Hkv * G, Hkv=Hkv, n_stream=n_stream, n_needles=0)
    q, k, v, sl, _ = configs.make_inputs(w, 5)
    n_mid = (w.T - w.n_stream - w.n_sink) // block
    starts = torch.full((Hkv, n_blocks), -1, dtype=torch.int32)
    for g in range(Hkv):
        pick = gen.distinct_ints(6, 100 + g, min(n_blocks, n_mid), n_mid).sort().values[:max(0, n_blocks - g)]
        starts[g, :len(pick)] = (w.n_sink + pick * block).to(torch.int32)
    qd, kd, vd, sld, bd = (t.cuda() for t in (q, k, v, sl, starts))
    L = ihip.Layer(qd, kd, sld, 1, w.n_sink, w.n_stream)
    need = L.workspace_bytes(ihip.OP_ATTN_DECODE, [block], [max(n_blocks, 1)])
    total = w.n_sink + n_blocks * block + n_stream
    coarse = Hkv * G * (-(-total // 256)) * 130 * 4
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream)
    got = []
    for size in (need, max(need - 1, coarse)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out, lse = L.sparse_attn_decode(qd, kd, vd, bd, block, want_lse=True, ws=ws)
        got.append(out.float().cpu())
        for g in range(Hkv):
            s = starts[g][starts[g] >= 0].numpy()
            ref, ref_lse = o.attend(0, g, 0, s, np.minimum(block, w.T - w.n_stream - s).astype(np.int32))
            assert np.abs(got[-1][0, g * G:(g + 1) * G].numpy() - ref).max() <= 4e-3, (size, g)
            np.testing.assert_allclose(lse[0, g * G:(g + 1) * G].cpu().numpy(), ref_lse, rtol=2e-5, atol=2e-5)
    assert (got[0] - got[1]).abs().max() <= 4e-3
    if need > coarse:
        small = torch.empty(Hkv * G * 130 * 4 // 2, dtype=torch.uint8, device="cuda")
        with pytest.raises(ihip.IhipError):
            L.sparse_attn_decode(qd, kd, vd, bd, block, ws=small)


def test_attention_splits_at_the_static_array(ihip):
    """A plan that fits the static scratch array with the coarse splits only: the reported bytes are the coarse ones, and the
    static call and the workspace call, with that much scratch or more, give identical bits."""
    B, Hkv, G, keep, limit = 2, 1, 8, 4096, 8 << 20
    q = torch.randn((B, Hkv * G, 1, 128), device="cuda").bfloat16()
    extra = B * Hkv * G * 130 * 4 * (55 - 21)             # 5,248 key slots: 55 fine splits, 21 coarse ones

    def layer(T):
        shape = torch.empty((B, Hkv, T, 0), dtype=torch.bfloat16)
        return ihip.Layer(q, shape, torch.full((B,), T, dtype=torch.int32, device="cuda"), 1, 128, 1024)

    T = 1 << 20
    while layer(T).workspace_bytes(ihip.OP_DECODE_LAYER, [1], [keep]) + extra // 2 > limit:      # a call more or less in the middle
        T -= 4096
    L = layer(T)
    need = L.workspace_bytes(ihip.OP_DECODE_LAYER, [1], [keep])
    assert need <= limit < need + extra
    k, v = (torch.randn((B, Hkv, T, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    outs = [torch.empty((B, Hkv * G, 1, 128), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    for size, out in ((need, outs[0]), (need + extra, outs[1])):
        L.decode_layer(q, k, v, [1], [keep], ws=torch.empty(size, dtype=torch.uint8, device="cuda"), out=out)
    L.decode_layer_static(q, k, v, [1], [keep], outs[2])
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    with pytest.raises(ihip.IhipError):
        L.decode_layer(q, k, v, [1], [keep], ws=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("B,T", [(3, 262144 + 512), (3, 262144 + 1568), (1, 294912 + 1000), (1, 294912 + 1500), (1, 393216 + 1000), (1, 393216 + 1500)])
@pytest.mark.parametrize("fp8,rope", [(False, False), (False, True), (True, True)])
def test_long_token_major_rows_score_as_head_major_ones(ihip, B, T, fp8, rope):
    """To either side of the lengths where the order of the grid changes; 8 KV heads, chunks for the vector and the matrix-core kernels."""
    Hq, Hkv = 32, 8
    g = torch.Generator(device="cuda").manual_seed(B * T + 2 * fp8 + rope)
    k = torch.randint(-3, 4, (B, T, Hkv, 128), generator=g, device="cuda", dtype=torch.int8)
    k = k.to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else k.to(torch.bfloat16)
    token_major, head_major = k.transpose(1, 2), k.transpose(1, 2).contiguous()
    q = torch.randint(-3, 4, (B, Hq, 1, 128), generator=g, device="cuda").to(torch.bfloat16)
    sl = torch.tensor([T, T - 70001, T - 131][:B], dtype=torch.int32, device="cuda")
    L = ihip.Layer(q, head_major, sl, 1, 128, 1024)
    kw = {"kv_scales": (1.0, 1.0)} if fp8 else {}
    if rope:
        cos, sin = gen.quarter_turn_table(16384, 128)
        kw["rope"] = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    for chunk in (128, 16):
        got = []
        for rows in (head_major, token_major):
            blocks = torch.empty((B * Hkv, 96), dtype=torch.int32, device="cuda")
            out = L.decode_layer(q, rows, rows, [chunk], [96], out_blocks=blocks, **kw)
            got.append((out, blocks))
        assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][0], got[1][0])
