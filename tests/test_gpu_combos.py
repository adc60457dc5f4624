"""GPU parity of the decode layer with several variants at once (dynamic RoPE,
FP8 K/V, paged K/V, all-heads pooling, mask caching) through
ihip_decode_layer_ex, against the CPU oracle.

Integer-valued inputs, the quarter-turn rotary table and power-of-two FP8
scales keep every score an exact integer multiple on both sides: kept block
lists are compared bit for bit, outputs within 2e-2."""
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


def scatter_to_pages(k, v, page, seed, fill, spare=5):
    """[B,Hkv,T,d] -> pools [n_pages,Hkv,page,d] with a seeded random page order + block table."""
    B, Hkv, T, d = k.shape
    per_seq = (T + page - 1) // page
    n_pages = B * per_seq + spare
    order = gen.distinct_ints(seed, 77, B * per_seq, n_pages).view(B, per_seq)
    k_pool = torch.full((n_pages, Hkv, page, d), fill, dtype=k.dtype)      # unused rows hold junk
    v_pool = torch.full((n_pages, Hkv, page, d), fill, dtype=v.dtype)
    pad = per_seq * page - T
    kp = torch.nn.functional.pad(k, (0, 0, 0, pad)).view(B, Hkv, per_seq, page, d)
    vp = torch.nn.functional.pad(v, (0, 0, 0, pad)).view(B, Hkv, per_seq, page, d)
    for b in range(B):
        k_pool[order[b]] = kp[b].permute(1, 0, 2, 3)
        v_pool[order[b]] = vp[b].permute(1, 0, 2, 3)
    return k_pool, v_pool, order.to(torch.int32)


class Case:
    """Inputs of one workload in every representation the variants need."""

    def __init__(self, ihip, orc, w, sl, rope, fp8, paged, prune_style="relative", seed=0):
        self.w = w
        q, k, v, _, _ = configs.make_inputs(w, seed, kind="int")
        self.q, self.sl = q, sl
        self.scales = (0.5, 0.25) if fp8 else None
        if fp8:       # values -2..2 over a power-of-two scale are E4M3 numbers: lossless
            k, v = gen.to_e4m3(k, self.scales[0]), gen.to_e4m3(v, self.scales[1])
        self.k, self.v = k, v
        self.cos, self.sin = gen.quarter_turn_table(w.T, w.d)
        self.rope_spec = orc.RopeSpec(self.cos.numpy(), self.sin.numpy(), prune=prune_style, attn="streaming") \
            if rope else None
        style = {"relative": ihip.ROPE_RELATIVE, "chunk": ihip.ROPE_CHUNK_INDEXED}[prune_style]
        self.rope = ihip.Rope(self.cos.cuda(), self.sin.cuda(), style, ihip.ROPE_STREAMING) if rope else None
        self.kd, self.vd = k.cuda(), v.cuda()
        self.paged = None
        if paged:
            k_pool, v_pool, table = scatter_to_pages(k, v, paged, seed=3, fill=7)
            self.paged = ihip.PagedKV(k_pool.cuda(), v_pool.cuda(), table.cuda())
        self.chunks = [s[0] for s in w.stages]
        self.keeps = [s[1] for s in w.stages]

    def oracle(self, orc, q=None, sl=None):
        return orc.Oracle(self.q if q is None else q, self.k, self.v, (self.sl if sl is None else sl).tolist(), 1,
                          self.w.n_sink, self.w.n_stream, rope=self.rope_spec, kv_scales=self.scales)

    def layer_kwargs(self):
        return dict(rope=self.rope, kv_scales=self.scales, paged=self.paged)


COMBOS = [
    dict(rope=True, fp8=True, paged=0),
    dict(rope=True, fp8=False, paged=16),
    dict(rope=False, fp8=True, paged=16),
    dict(rope=True, fp8=True, paged=64),
    dict(rope=True, fp8=True, paged=16, prune_style="chunk"),
]


@pytest.mark.parametrize("combo", COMBOS, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()))
@pytest.mark.parametrize("T,B", [(8192, 1), (4096 + 37, 2)])
def test_combined_variants_match_the_oracle(ihip, orc, combo, T, B):
    w = configs.shrink(configs.CFG1, T=T, B=B, n_needles=0)
    sl = torch.tensor([T, T - 1001][:B], dtype=torch.int32)
    c = Case(ihip, orc, w, sl, **combo)
    qd, sld = c.q.cuda(), sl.cuda()
    L = ihip.Layer(qd, c.kd, sld, 1, w.n_sink, w.n_stream)
    P = w.B * w.Hkv
    blocks = torch.empty((P, c.keeps[-1]), dtype=torch.int32, device="cuda")
    out = L.decode_layer(qd, c.kd, c.vd, c.chunks, c.keeps, out_blocks=blocks, **c.layer_kwargs())
    torch.cuda.synchronize()
    o = c.oracle(orc)
    for b in range(B):
        for g in range(w.Hkv):
            pr = o.prune(b, g, 0, w.stages)
            kp = blocks[b * w.Hkv + g].cpu().numpy()
            assert np.array_equal(kp[kp >= 0], pr.block_starts), (b, g)
            ref, _ = o.attend(b, g, 0, pr.block_starts, pr.block_lens)
            got = out[b, g * w.G:(g + 1) * w.G, 0].float().cpu().numpy()
            assert np.abs(got - ref[:, 0]).max() <= 2e-2, (b, g)


def test_all_heads_pooling_with_rope_and_pages(ihip, orc):
    w = configs.shrink(configs.CFG1, T=4096, n_needles=0)
    sl = torch.tensor([4096], dtype=torch.int32)
    c = Case(ihip, orc, w, sl, rope=True, fp8=False, paged=16)
    qd = c.q.cuda()
    L = ihip.Layer(qd, c.kd, sl.cuda(), 1, w.n_sink, w.n_stream)
    blocks = torch.empty((w.Hkv, c.keeps[-1]), dtype=torch.int32, device="cuda")
    out = L.decode_layer(qd, None, None, c.chunks, c.keeps, out_blocks=blocks, pooling=ihip.POOL_ALL_HEADS,
                         **c.layer_kwargs())
    torch.cuda.synchronize()
    o = c.oracle(orc)
    prs = o.prune_all_heads(0, 0, w.stages)
    for g in range(w.Hkv):
        kp = blocks[g].cpu().numpy()
        assert np.array_equal(kp[kp >= 0], prs[g].block_starts), g
        ref, _ = o.attend(0, g, 0, prs[g].block_starts, prs[g].block_lens)
        got = out[0, g * w.G:(g + 1) * w.G, 0].float().cpu().numpy()
        assert np.abs(got - ref[:, 0]).max() <= 2e-2


@pytest.mark.parametrize("combo", [dict(rope=True, fp8=False, paged=0), dict(rope=True, fp8=True, paged=16)],
                         ids=["rope", "rope-fp8-paged"])
def test_mask_caching_with_variants_follows_oracle(ihip, orc, combo):
    # Alg. 4's refresh schedule on top of the variants: sequences grow, queries change every step
    refresh = (4, 2, 1)
    w = configs.shrink(configs.CFG1, B=2, Hq=8, Hkv=2, T=3000, n_stream=256, n_needles=0,
                       stages=((64, 8), (16, 8), (4, 16)))
    lens0 = [2900, 2200]
    c = Case(ihip, orc, w, torch.tensor(lens0, dtype=torch.int32), **combo)
    state = None
    cached = {(b, g): [np.zeros(0, np.int64)] * 3 for b in range(w.B) for g in range(w.Hkv)}
    P = w.B * w.Hkv
    for step in range(9):
        sl = torch.tensor([lens0[0] + step, lens0[1] + 3 * step], dtype=torch.int32)
        q = configs.make_q(w, 100 + step, kind="int")
        qd, sld = q.cuda(), sl.cuda()
        L = ihip.Layer(qd, c.kd, sld, 1, w.n_sink, w.n_stream)
        if state is None:
            state = L.mask_state(c.keeps)
        first = ihip.first_stage_due(step, refresh)
        out = L.decode_layer(qd, c.kd, c.vd, c.chunks, c.keeps, stage_starts=state, first_stage=first,
                             **c.layer_kwargs())
        torch.cuda.synchronize()
        o = c.oracle(orc, q=q, sl=sl)
        off, st_gpu = 0, []
        for keep in c.keeps:
            st_gpu.append(state[off:off + P * keep].view(P, keep).cpu().numpy())
            off += P * keep
        for b in range(w.B):
            for g in range(w.Hkv):
                kept, bs, bl = o.prune_from(b, g, 0, w.stages, first, cached[(b, g)])
                cached[(b, g)] = kept
                p = b * w.Hkv + g
                for i in range(3):
                    got = st_gpu[i][p]
                    assert got[got >= 0].tolist() == kept[i].tolist(), (step, b, g, i)
                ref, _ = o.attend(b, g, 0, bs, bl)
                err = np.abs(out[b, g * w.G:(g + 1) * w.G, 0].float().cpu().numpy() - ref[:, 0]).max()
                assert err <= 2e-2, (step, b, g, err)


@pytest.mark.parametrize("T", [2048, 4096 + 37])
def test_keep_everything_with_all_variants_is_rotary_attention(ihip, T):
    # Every chunk kept: the decode layer with streaming RoPE over FP8 pages must be ordinary rotary
    # attention of the last token over the dequantised K and V (torch, fp64; no oracle involved).
    w = configs.shrink(configs.CFG1, T=T, B=2, n_needles=0)
    n1 = (T - w.n_sink - w.n_stream + 63) // 64
    stages = ((64, n1), (16, 4 * n1), (4, 16 * n1))
    q, k, v, _, _ = configs.make_inputs(w, 4)
    sl = torch.tensor([T, T - 300], dtype=torch.int32)
    scales = (1.0 / 32, 1.0 / 16)
    k8, v8 = gen.to_e4m3(k, scales[0]), gen.to_e4m3(v, scales[1])
    kf = k8.view(torch.float8_e4m3fn).double() * scales[0]
    vf = v8.view(torch.float8_e4m3fn).double() * scales[1]
    cos, sin = gen.rope_table(T + 64, w.d)
    k_pool, v_pool, table = scatter_to_pages(k8, v8, 16, seed=11, fill=3)
    pg = ihip.PagedKV(k_pool.cuda(), v_pool.cuda(), table.cuda())
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    qd = q.cuda()
    L = ihip.Layer(qd, k8.cuda(), sl.cuda(), 1, w.n_sink, w.n_stream)
    out = L.decode_layer(qd, None, None, [s[0] for s in stages], [s[1] for s in stages], rope=rp, kv_scales=scales,
                         paged=pg)
    torch.cuda.synchronize()
    G, d = w.G, w.d
    for b in range(w.B):
        n = int(sl[b])
        pos = torch.arange(n)
        c, s_ = cos[pos].double(), sin[pos].double()
        ke, ko = kf[b, :, :n, 0::2], kf[b, :, :n, 1::2]
        kr = torch.empty((w.Hkv, n, d), dtype=torch.float64)
        kr[..., 0::2], kr[..., 1::2] = ke * c - ko * s_, ke * s_ + ko * c
        qe, qo = q[b, :, 0, 0::2].double(), q[b, :, 0, 1::2].double()
        qr = torch.empty((w.Hq, d), dtype=torch.float64)
        qr[:, 0::2] = qe * c[n - 1] - qo * s_[n - 1]
        qr[:, 1::2] = qe * s_[n - 1] + qo * c[n - 1]
        logits = torch.einsum("hd,hnd->hn", qr, kr.repeat_interleave(G, 0)) / d ** 0.5
        ref = torch.einsum("hn,hnd->hd", torch.softmax(logits, -1), vf[b, :, :n].repeat_interleave(G, 0))
        assert (out[b, :, 0].cpu().double() - ref).abs().max().item() <= 2e-2, b


# Shapes whose stages run on the matrix cores (4 or 8 heads per group, workgroups enough for the compute units), at the edges of
# those kernels: chunks of 1, 2, 4, 8, 16 and 32 keys, a chunk cut short at the end of the middle range, a last wave that is partly
# empty, kept lists with holes, more pages per chunk than a wave keeps, K rows further apart than 32-bit offsets reach.
TILE_CASES = [
    dict(G=8, Hkv=2, B=1, T=52003, stages=((8, 6144), (4, 512)), rope=False, fp8=False, paged=0),
    dict(G=8, Hkv=4, B=1, T=52003, stages=((8, 6144), (4, 512)), rope=True, fp8=False, paged=0),
    dict(G=8, Hkv=4, B=1, T=52003, stages=((8, 6144), (4, 512)), rope=True, fp8=False, paged=0, far=True),
    dict(G=8, Hkv=2, B=1, T=52003, stages=((8, 6144), (4, 512)), rope=False, fp8=True, paged=0),
    dict(G=8, Hkv=4, B=1, T=52003, stages=((8, 6144), (4, 512)), rope=True, fp8=True, paged=16),
    dict(G=8, Hkv=1, B=2, T=110003, stages=((32, 1024), (4, 256)), rope=False, fp8=False, paged=1),
    dict(G=4, Hkv=2, B=2, T=67003, stages=((32, 1024), (2, 256)), rope=False, fp8=True, paged=1),
    dict(G=4, Hkv=4, B=2, T=76003, stages=((16, 4096), (2, 512)), rope=False, fp8=False, paged=4),
    dict(G=4, Hkv=8, B=1, T=51003, stages=((8, 6144), (4, 3072), (1, 500)), rope=True, fp8=True, paged=64),
    dict(G=4, Hkv=4, B=1, T=51003, stages=((8, 6144), (1, 500)), rope=False, fp8=True, paged=0),
    dict(G=4, Hkv=8, B=1, T=51003, stages=((8, 6144), (4, 3072)), rope=True, fp8=False, paged=16),
    dict(G=4, Hkv=8, B=1, T=51003, stages=((8, 6144), (4, 3072), (1, 500)), rope=True, fp8=False, paged=0),
]


@pytest.mark.parametrize("c", TILE_CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items() if k != "stages"))
def test_matrix_core_decode_stages(ihip, orc, c):
    w = configs.shrink(configs.CFG1, T=c["T"], B=c["B"], Hq=c["Hkv"] * c["G"], Hkv=c["Hkv"], stages=c["stages"], n_needles=0)
    sl = torch.tensor([w.T, w.T - 1001][:w.B], dtype=torch.int32)
    case = Case(ihip, orc, w, sl, c["rope"], c["fp8"], c["paged"])
    kd = case.kd
    if c.get("far"):              # one token every 84 KB: the slab is 4.4 GB long
        far = torch.empty((w.T, 42000), dtype=torch.bfloat16, device="cuda")
        view = far[:, :w.Hkv * w.d].view(w.T, w.Hkv, w.d).permute(1, 0, 2).unsqueeze(0)
        view.copy_(kd)
        kd = view
    qd, sld = case.q.cuda(), sl.cuda()
    L = ihip.Layer(qd, kd, sld, 1, w.n_sink, w.n_stream)
    blocks = torch.empty((L.P, case.keeps[-1]), dtype=torch.int32, device="cuda")
    L.decode_layer(qd, kd, case.vd, case.chunks, case.keeps, out_blocks=blocks, **case.layer_kwargs())
    o = case.oracle(orc)
    prs = {}
    for b in range(w.B):
        for g in range(w.Hkv):
            prs[b, g] = o.prune(b, g, 0, w.stages)
            kp = blocks[b * w.Hkv + g].cpu().numpy()
            assert np.array_equal(kp[kp >= 0], prs[b, g].block_starts), (b, g)
    if c["rope"] + c["fp8"] + bool(c["paged"]) > 1:
        return                    # the single-stage call takes one variant at a time
    # scores and representatives of every stage, which the layer call does not return
    variant = dict(rope=case.rope, k_scale=case.scales[0] if c["fp8"] else None, paged=case.paged)
    parents, pchunk = None, 0
    for i, (l_c, keep) in enumerate(w.stages):
        scores, rep = L.prune_stage(qd, kd, l_c, parents, pchunk, want_rep=True, **variant)
        parents, pchunk = L.select_blocks(scores, l_c, keep, parents, pchunk), l_c
        for (b, g), pr in prs.items():
            st = pr.stages[i]
            n, p = len(st.starts), b * w.Hkv + g
            assert np.array_equal(scores[p, :n].cpu().numpy(), st.scores) and torch.isneginf(scores[p, n:]).all(), (b, g, i)
            rp = rep[b, g * w.G:(g + 1) * w.G, 0].cpu().numpy()
            assert np.array_equal(rp[:, :n], st.reps) and (rp[:, n:] == -1).all(), (b, g, i)


@pytest.mark.parametrize("G,Hkv,stages", [(4, 8, ((8, 6144), (4, 512))), (8, 4, ((8, 6144), (4, 512)))], ids=["g4", "g8"])
def test_matrix_core_decode_rotates_to_fp32(ihip, orc, G, Hkv, stages):
    """Relative style on a real rotary table: the rotated queries are three bf16 operands (value, rest, rest of the rest).
    Against the score of the kernel's own representative in 64 bits, RMS over N(0,1) rows: 128 fp32 sums of about 11 give 4e-6,
    without the last operand (2^-18 of every query element) it is 2.9e-5, without the second 1.9e-2.  The searches against
    the fp32 oracle: near ties, within 1e-4 of a difference that has standard deviation 16, are 1e-5 of the six comparisons
    of 8 keys at most."""
    w = configs.shrink(configs.CFG1, T=51003, B=1, Hq=Hkv * G, Hkv=Hkv, stages=stages, n_needles=0)
    q, k, v, sl, _ = configs.make_inputs(w, 8)
    cos, sin = gen.rope_table(w.n_stream + 2, w.d)
    o = orc.Oracle(q, k, v, sl.tolist(), 1, w.n_sink, w.n_stream, rope=orc.RopeSpec(cos.numpy(), sin.numpy(), prune="relative"))
    qd, kd = q.cuda(), k.cuda()
    L = ihip.Layer(qd, kd, sl.cuda(), 1, w.n_sink, w.n_stream)
    rope = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_NONE)
    prs = [o.prune(0, g, 0, stages) for g in range(Hkv)]
    c, s = cos[w.n_stream].double().cuda(), sin[w.n_stream].double().cuda()
    x = qd[0, :, 0].double()
    qr = torch.stack((x[:, 0::2] * c - x[:, 1::2] * s, x[:, 0::2] * s + x[:, 1::2] * c), dim=-1).flatten(1)
    parents, pchunk = None, 0
    for i, (l_c, keep) in enumerate(stages):
        scores, rep = L.prune_stage(qd, kd, l_c, parents, pchunk, want_rep=True, rope=rope)
        flips = total = 0
        for g in range(Hkv):
            st = prs[g].stages[i]
            n, heads = len(st.starts), slice(g * G, (g + 1) * G)
            r = rep[0, heads, 0, :n].long()
            exact = torch.stack([(kd[0, g][r[h]].double() * qr[g * G + h]).sum(-1) for h in range(G)]).amax(0)
            err = scores[g, :n].double() - exact
            assert err.pow(2).mean().sqrt().item() <= 1e-5 and err.abs().max().item() <= 1e-4, (i, g)
            flips += (r.cpu().numpy() != st.reps).sum()
            total += r.numel()
        assert flips <= 1e-4 * total, (i, flips, total)
        starts = np.full((Hkv, keep), -1, np.int32)          # the oracle's list, so that the stages stay comparable
        for g in range(Hkv):
            starts[g, :len(prs[g].stages[i].kept_starts)] = prs[g].stages[i].kept_starts
        parents, pchunk = torch.from_numpy(starts).cuda(), l_c


# Batches with idle places (no keys) and sequences that end before their middle range.
IDLE_CASES = [
    dict(G=4, Hkv=2, T=9003, stages=((16, 128), (4, 64)), rope=True, fp8=False, paged=0),
    dict(G=4, Hkv=2, T=9003, stages=((16, 128), (4, 64)), rope=True, fp8=False, paged=16, prune_style="chunk"),
    dict(G=1, Hkv=2, T=9003, stages=((16, 128), (4, 64)), rope=False, fp8=True, paged=16),
    # large enough for the matrix-core kernels
    dict(G=8, Hkv=2, T=52003, stages=((8, 6144), (4, 512)), rope=True, fp8=False, paged=16),
    dict(G=4, Hkv=4, T=51003, stages=((8, 6144), (4, 512)), rope=False, fp8=True, paged=16),
    dict(G=4, Hkv=4, T=51003, stages=((8, 6144), (4, 512)), rope=True, fp8=True, paged=0),
]


@pytest.mark.parametrize("c", IDLE_CASES, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items() if k != "stages"))
def test_idle_and_short_sequences_in_a_decode_batch(ihip, orc, c):
    """Every key and every page behind a sequence's length holds NaN (block-table entries there name such pages):
    nothing of it may reach another sequence, a sequence without chunks keeps no block, one without keys reads none."""
    w = configs.shrink(configs.CFG1, T=c["T"], B=4, Hq=c["Hkv"] * c["G"], Hkv=c["Hkv"], stages=c["stages"], n_needles=0)
    sl = torch.tensor([0, w.T, w.n_sink + w.n_stream - 1, w.T - 1001], dtype=torch.int32)
    case = Case(ihip, orc, w, sl, c["rope"], c["fp8"], c["paged"], prune_style=c.get("prune_style", "relative"))
    nan = 0x7f if c["fp8"] else float("nan")
    for b, n in enumerate(sl.tolist()):
        case.kd[b, :, n:] = nan
        case.vd[b, :, n:] = nan
        if case.paged is not None:
            behind = case.paged.block_table[b, -(-n // c["paged"]):].long()
            case.paged.k_pool[behind] = nan
            case.paged.v_pool[behind] = nan
    qd = case.q.cuda()
    L = ihip.Layer(qd, case.kd, sl.cuda(), 1, w.n_sink, w.n_stream)
    blocks = torch.empty((L.P, case.keeps[-1]), dtype=torch.int32, device="cuda")
    out = L.decode_layer(qd, case.kd, case.vd, case.chunks, case.keeps, out_blocks=blocks, **case.layer_kwargs())
    torch.cuda.synchronize()
    o = case.oracle(orc)
    for b in range(w.B):
        for g in range(w.Hkv):
            kp = blocks[b * w.Hkv + g].cpu().numpy()
            if b in (0, 2):
                assert (kp == -1).all(), (b, g)
            if b == 0:
                continue
            pr = o.prune(b, g, 0, w.stages)
            assert np.array_equal(kp[kp >= 0], pr.block_starts), (b, g)
            ref, _ = o.attend(b, g, 0, pr.block_starts, pr.block_lens)
            assert np.abs(out[b, g * w.G:(g + 1) * w.G, 0].float().cpu().numpy() - ref[:, 0]).max() <= 2e-2, (b, g)
