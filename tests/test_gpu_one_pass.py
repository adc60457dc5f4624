"""Decode plans whose stages are scored in one pass over the middle range (prune_decode_nest.h, select_chain.hip) against the
stage-by-stage kernels.  The same call takes the one or the other by its workspace: the scores of the one pass come last, and a
byte less than ihip_workspace_bytes says leaves no room for them.  Inputs are whole numbers (and quarter turns), so every
score is exact in both and the lists and outputs have to be the same bits, ties included.  With N(0,1) inputs the list is
compared with an exact selection among the scores that the one pass left in its workspace."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


def _kernels(ihip, run):
    """Launches of the pruning and of the selection kernels in one call."""
    ihip.profile_read()
    ihip.profile_enable(True)
    try:
        run()
    finally:
        ihip.profile_enable(False)
    launches = {name: n for name, (_, n) in ihip.profile_read().items()}
    return tuple(sum(n for name, n in launches.items() if name.startswith(kind)) for kind in ("prune_decode", "select_blocks"))


def _case(ihip, Hq, Hkv, lens, stages, fmt, rope, spread=3, n_sink=64, n_stream=256, pooling=None, seed=0):
    g = torch.Generator().manual_seed(seed)
    B, T, D = len(lens), max(lens), 128
    whole = lambda *shape: torch.randint(-spread, spread + 1, shape, generator=g).float()
    q, k, v = whole(B, Hq, 1, D).bfloat16().cuda(), whole(B, Hkv, T, D), whole(B, Hkv, T, D)
    kw = {}
    if "fp8" in fmt:
        k, v = (t.to(torch.float8_e4m3fn).view(torch.uint8) for t in (k, v))
        kw["kv_scales"] = (1.0, 1.0)
    else:
        k, v = k.bfloat16(), v.bfloat16()
    k, v = k.cuda(), v.cuda()
    if "paged" in fmt:
        page = 16
        n = -(-T // page)
        order = torch.randperm(B * n, generator=g).cuda()
        pools = []
        for t in (k, v):
            full = torch.zeros((B, Hkv, n * page, D), dtype=t.dtype, device="cuda")
            full[:, :, :T] = t
            pool = torch.empty((B * n, Hkv, page, D), dtype=t.dtype, device="cuda")
            pool[order] = full.view(B, Hkv, n, page, D).permute(0, 2, 1, 3, 4).reshape(B * n, Hkv, page, D)
            pools.append(pool)
        kw["paged"] = ihip.binding.PagedKV(pools[0], pools[1], order.to(torch.int32).view(B, n).contiguous())
    if rope:
        turn = torch.arange(T + n_sink + n_stream + stages[-1][0] * stages[-1][1]) % 4          # quarter turns: cos and sin are 0 and +-1
        c = torch.tensor([1.0, 0.0, -1.0, 0.0])[turn].view(-1, 1).repeat(1, D // 2).contiguous().cuda()
        s = torch.tensor([0.0, 1.0, 0.0, -1.0])[turn].view(-1, 1).repeat(1, D // 2).contiguous().cuda()
        kw["rope"] = ihip.binding.Rope(c, s, ihip.binding.ROPE_RELATIVE, ihip.binding.ROPE_STREAMING)
    if pooling:
        kw["pooling"] = ihip.binding.POOL_ALL_HEADS
    chunks, keeps = [s[0] for s in stages], [s[1] for s in stages]
    shape = torch.empty((B, Hkv, T, 0), dtype=torch.bfloat16)
    L = ihip.Layer(q, shape, torch.tensor(lens, dtype=torch.int32, device="cuda"), 1, n_sink, n_stream)
    need = L.workspace_bytes(ihip.OP_DECODE_LAYER, chunks, keeps)
    got = []
    for size, launches in ((need, (1, 1)), (need - 1, (len(stages), len(stages)))):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
        lse = torch.empty((B, Hq), dtype=torch.float32, device="cuda")
        out = torch.empty((B, Hq, 1, D), dtype=torch.bfloat16, device="cuda")
        assert _kernels(ihip, lambda: L.decode_layer(q, k, v, chunks, keeps, ws=ws, out=out, out_blocks=blocks, lse=lse, **kw)) == launches
        got.append((out.cpu(), lse.cpu(), blocks.cpu()))
    assert torch.equal(got[0][2], got[1][2])
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1])
    return got[0][2]


THREE = ((64, 12), (16, 20), (4, 40))


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "paged", "fp8-paged"])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (64, 8), (6, 3), (4, 4)])
def test_storage_rope_and_groups(ihip, Hq, Hkv, fmt, rope):
    _case(ihip, Hq, Hkv, [2405, 1501], THREE, fmt, rope)


@pytest.mark.parametrize("stages", [
    ((256, 5), (16, 30), (4, 60)), ((128, 9), (32, 17), (8, 33)), ((32, 50), (4, 100)), ((16, 64), (8, 65)), ((8, 200), (4, 200)),
    ((256, 6), (64, 12), (16, 24), (4, 48)), ((64, 512), (16, 512), (4, 512)), ((64, 1), (4, 1)),
], ids=lambda s: "-".join("%d:%d" % x for x in s))
@pytest.mark.parametrize("T", [4099, 5000, 400])
def test_plans_and_lengths(ihip, stages, T):
    """400: the middle range is shorter than a wave's 64 keys; the last chunk is cut short at 79 and 4 keys past a multiple of 256."""
    _case(ihip, 8, 2, [T], stages, "bf16", T == 5000)


def test_ragged_batch_with_idle_places(ihip):
    """Sequences shorter than sink and window, and an empty place: their lists are empty."""
    lens = [3000, 320, 1, 0, 321, 700]
    blocks = _case(ihip, 32, 8, lens, THREE, "bf16", False)
    for b, T in enumerate(lens):
        assert (blocks.view(len(lens), 8, -1)[b] >= 0).any() == (T > 320), (b, T)
    _case(ihip, 32, 8, lens, THREE, "fp8-paged", True)


def test_pooled_over_all_heads(ihip):
    blocks = _case(ihip, 16, 4, [2000, 1200], THREE, "bf16", False, pooling=True)
    assert (blocks.view(2, 4, -1) == blocks.view(2, 4, -1)[:, :1]).all()


def test_heavy_ties(ihip):
    """All scores equal (more candidates in one bin than threads): the lowest positions are kept."""
    blocks = _case(ihip, 8, 2, [9000], ((8, 800), (4, 900)), "bf16", False, spread=0)
    assert torch.equal(blocks[0], 64 + 4 * torch.arange(900, dtype=torch.int32))


# candidates of a selection on either side of the steps from one to two and four per thread, and the most of the two (2,048)
SIZES = [(1, 512, ((8, 256), (4, 200))), (2, 513, ((8, 257), (4, 200))), (3, 1024, ((8, 512), (4, 300))), (4, 1025, ((8, 513), (4, 300))),
         (5, 1500, ((8, 750), (4, 1001))), (6, 2048, ((8, 1024), (4, 700))), (7, 600, ((64, 512), (16, 512), (4, 512))), (8, 375, ((16, 375), (4, 1400)))]


def _length(n_slots, stages):                    # the middle range ends inside its last chunk
    return 64 + 256 + (n_slots - 1) * stages[0][0] + stages[0][0] // 2 + 1


@pytest.mark.parametrize("seed,n_slots,stages", SIZES, ids=lambda x: None if isinstance(x, tuple) else str(x))
def test_selection_sizes(ihip, seed, n_slots, stages):
    """Scores that hardly ever tie: whole numbers up to 100 in the inputs, exact sums far below 2^24."""
    _case(ihip, 8, 2, [_length(n_slots, stages)], stages, "bf16", False, spread=100, seed=seed)


@pytest.mark.parametrize("seed,n_slots,stages", SIZES + [(9, 300, ((64, 64), (16, 128), (4, 128)))],
                         ids=lambda x: None if isinstance(x, tuple) else str(x))
@pytest.mark.parametrize("G", [4, 8])
def test_lists_are_the_best_of_the_scores(ihip, G, seed, n_slots, stages):
    """N(0,1) inputs, two sequences of unlike lengths: the list is the exact choice, stage by stage, among the scores of the pass."""
    n_sink, n_stream, Hkv = 64, 256, 2
    lens = [_length(n_slots, stages), max(400, _length(n_slots, stages) * 5 // 8)]
    g = torch.Generator().manual_seed(seed)
    q = torch.randn((2, Hkv * G, 1, 128), generator=g).bfloat16().cuda()
    k, v = (torch.randn((2, Hkv, lens[0], 128), generator=g).bfloat16().cuda() for _ in range(2))
    chunks, keeps = [s[0] for s in stages], [s[1] for s in stages]
    L = ihip.Layer(q, k, torch.tensor(lens, dtype=torch.int32, device="cuda"), 1, n_sink, n_stream)
    ws = torch.full((L.workspace_bytes(ihip.OP_DECODE_LAYER, chunks, keeps),), 0xA5, dtype=torch.uint8, device="cuda")
    blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
    assert _kernels(ihip, lambda: L.decode_layer(q, k, v, chunks, keeps, ws=ws, out_blocks=blocks)) == (1, 1)
    # the scores come last: a problem's stages one after the other, each rounded up to 64
    n = [n_slots * (chunks[0] // c) for c in chunks]
    stride = sum((x + 63) // 64 * 64 for x in n)
    nbytes = L.P * stride * 4
    at = ws.numel() - (nbytes + 255) // 256 * 256
    scores = ws[at:at + nbytes].view(torch.float32).view(L.P, stride).cpu().numpy()
    for p in range(L.P):
        kept, first, lo = None, 0, n_sink
        hi = lens[p // Hkv] - n_stream
        for i, (c, keep) in enumerate(stages):
            ratio = chunks[i - 1] // c if i else 1
            cand = np.arange(n[0]) if i == 0 else (kept[:, None] * ratio + np.arange(ratio)).ravel()
            s = scores[p, first + cand]
            there = lo + cand * c < hi
            assert np.isfinite(s[there]).all() and (s[~there] == -np.inf).all()
            cand, s = cand[there], s[there]
            kept = np.sort(cand[np.lexsort((cand, -s))[:keep]])
            first += (n[i] + 63) // 64 * 64
        want = np.full(keeps[-1], -1)
        want[:len(kept)] = lo + kept * chunks[-1]
        assert (blocks[p].cpu().numpy() == want).all(), p


def test_several_single_query_blocks(ihip):
    """ihip_prune_all with Tq = 3, b_q = 1 (a problem per query): every query's list is that of a call for it alone."""
    g = torch.Generator().manual_seed(1)
    T, chunks, keeps = 3000, [64, 16], [12, 20]
    q, k = (torch.randint(-3, 4, s, generator=g).bfloat16().cuda() for s in ((2, 8, 3, 128), (2, 2, T, 128)))
    layer = lambda x, back: ihip.Layer(x, k, torch.tensor([T - back, T - 700 - back], dtype=torch.int32, device="cuda"), 1, 64, 256)  # noqa: E731
    got = layer(q, 0).prune_all(q, k, chunks, keeps).view(2, 2, 3, -1)
    for t in range(3):
        one = q[:, :, t:t + 1].contiguous()
        assert torch.equal(got[:, :, t], layer(one, 2 - t).prune_all(one, k, chunks, keeps).view(2, 2, -1)), t


@pytest.mark.parametrize("Hq,Hkv,B,T,fmt,rope,stages,one_pass", [
    (32, 8, 1, 32768, "bf16", False, ((64, 64), (16, 64), (4, 128)), True),
    (8, 8, 1, 32768, "bf16", False, ((32, 50), (4, 100)), False),          # two stages, one head a group: the searches read few rows
    (8, 8, 4, 16384, "fp8", True, ((32, 50), (4, 100)), False),
    (64, 8, 4, 16384, "fp8", True, ((64, 96), (8, 200)), True),            # eight heads: they read most of them
    (32, 8, 2, 131072, "bf16", False, ((64, 64), (16, 64), (4, 128)), False),
], ids=["4-heads", "1-head", "1-head-fp8-rope", "8-heads-fp8-rope", "long"])
def test_which_plans_go_in_one_pass(ihip, Hq, Hkv, B, T, fmt, rope, stages, one_pass):
    """Either way the lists of a batch of equal sequences are equal."""
    g = torch.Generator(device="cuda").manual_seed(2)
    q = torch.randn((1, Hq, 1, 128), generator=g, device="cuda").bfloat16().expand(B, -1, -1, -1).contiguous()
    k = torch.randn((1, Hkv, T, 128), generator=g, device="cuda").bfloat16()
    kw = {}
    if fmt == "fp8":
        k, kw["kv_scales"] = k.to(torch.float8_e4m3fn).view(torch.uint8), (1.0, 1.0)
    k = k.expand(B, -1, -1, -1).contiguous()
    if rope:
        kw["rope"] = ihip.Rope(torch.ones(4096, 64).cuda(), torch.zeros(4096, 64).cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    chunks, keeps = [s[0] for s in stages], [s[1] for s in stages]
    L = ihip.Layer(q, k, torch.full((B,), T, dtype=torch.int32, device="cuda"), 1, 128, 1024)
    blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
    n = 1 if one_pass else len(stages)
    assert _kernels(ihip, lambda: L.decode_layer(q, k, k, chunks, keeps, out_blocks=blocks, **kw)) == (n, n)
    assert (blocks.view(B, -1) == blocks.view(B, -1)[:1]).all() and (blocks >= 0).all()
