"""Decode plans whose last two stages are scored together from the keys of the chunks kept before them (prune_decode_nest.h with
parents, select_chain.hip), against the stage-by-stage kernels: the same call takes the one or the other by its workspace, whose
last bytes are the scores taken together.  Inputs are whole numbers (and quarter turns), so every score is exact in both and lists and
outputs have to be the same bits, ties included."""
import pytest
import torch

pytestmark = pytest.mark.gpu
D = 128


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


def _launches(ihip, run):
    ihip.profile_read()
    ihip.profile_enable(True)
    try:
        run()
    finally:
        ihip.profile_enable(False)
    return sum(n for name, (_, n) in ihip.profile_read().items() if name.startswith("prune_decode"))


def _inputs(ihip, Hq, Hkv, lens, fmt, rope, n_pos, seed=0, page=16):
    g = torch.Generator().manual_seed(seed)
    B, T = len(lens), max(lens)
    whole = lambda *shape: torch.randint(-3, 4, shape, generator=g).float()  # noqa: E731
    q, k, v = whole(B, Hq, 1, D).bfloat16().cuda(), whole(B, Hkv, T, D), whole(B, Hkv, T, D)
    kw = {}
    if "fp8" in fmt:
        k, v = (t.to(torch.float8_e4m3fn).view(torch.uint8) for t in (k, v))
        kw["kv_scales"] = (1.0, 1.0)
    else:
        k, v = k.bfloat16(), v.bfloat16()
    k, v = k.cuda(), v.cuda()
    if "paged" in fmt:
        n = -(-T // page)
        order = torch.randperm(B * n, generator=g).cuda()
        pools = []
        for t in (k, v):
            full = torch.zeros((B, Hkv, n * page, D), dtype=t.dtype, device="cuda")
            full[:, :, :T] = t
            pool = torch.empty((B * n, Hkv, page, D), dtype=t.dtype, device="cuda")
            pool[order] = full.view(B, Hkv, n, page, D).permute(0, 2, 1, 3, 4).reshape(B * n, Hkv, page, D)
            pools.append(pool)
        kw["paged"] = ihip.PagedKV(pools[0], pools[1], order.to(torch.int32).view(B, n).contiguous())
    if rope:
        turn = torch.arange(n_pos) % 4                # quarter turns: cos and sin are 0 and +-1
        c = torch.tensor([1.0, 0.0, -1.0, 0.0])[turn].view(-1, 1).repeat(1, D // 2).contiguous().cuda()
        s = torch.tensor([0.0, 1.0, 0.0, -1.0])[turn].view(-1, 1).repeat(1, D // 2).contiguous().cuda()
        kw["rope"] = ihip.Rope(c, s, ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    return q, k, v, kw


def _check(ihip, Hq, Hkv, lens, stages, fmt="bf16", rope=False, n_sink=64, n_stream=256, pooling=False, seed=0):
    B, T = len(lens), max(lens)
    chunks, keeps = [s[0] for s in stages], [s[1] for s in stages]
    q, k, v, kw = _inputs(ihip, Hq, Hkv, lens, fmt, rope, n_sink + n_stream + chunks[-1] * keeps[-1] + 8, seed)
    if pooling:
        kw["pooling"] = ihip.POOL_ALL_HEADS
    L = ihip.Layer(q, torch.empty((B, Hkv, T, 0), dtype=torch.bfloat16), torch.tensor(lens, dtype=torch.int32, device="cuda"), 1, n_sink, n_stream)
    need = L.workspace_bytes(ihip.OP_DECODE_LAYER, chunks, keeps)
    got = []
    for size, launches in ((need, len(stages) - 1), (need - 1, len(stages))):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
        out, lse = torch.empty((B, Hq, 1, D), dtype=torch.bfloat16, device="cuda"), torch.empty((B, Hq), device="cuda")
        assert _launches(ihip, lambda: L.decode_layer(q, k, v, chunks, keeps, ws=ws, out=out, out_blocks=blocks, lse=lse, **kw)) == launches
        got.append((blocks.cpu(), out.cpu().view(torch.int16), lse.cpu().view(torch.int32)))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    return got[0][0]


PLAN = ((64, 40), (16, 80), (4, 100))                 # 160 candidates of 16 keys, half of them kept


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "paged", "fp8-paged"])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (16, 2)])
def test_storage_rope_and_groups(ihip, Hq, Hkv, fmt, rope):
    _check(ihip, Hq, Hkv, [150003, 99001], PLAN, fmt, rope)


@pytest.mark.parametrize("stages", [
    ((256, 9), (64, 24), (16, 60), (4, 61)), ((128, 40), (32, 130), (8, 300)), ((64, 1), (16, 4), (4, 9)), ((64, 512), (16, 512), (4, 512)),
    ((128, 256), (16, 1024), (8, 900)), ((64, 3), (64, 3), (4, 30)),
], ids=lambda s: "-".join("%d:%d" % x for x in s))
def test_plans(ihip, stages):
    """Two and more chunks a parent, as large as the parent, up to 2,048 candidates; fewer kept than asked for."""
    _check(ihip, 16, 2, [140007], stages, seed=len(stages))


def test_ragged_batch_with_idle_places_and_cut_chunks(ihip):
    """Lists with places that hold no chunk, parents cut short by the end of the middle range, sequences without any."""
    lens = [150000, 64 + 256 + 64 * 20 + 7, 64 + 256 + 1, 300, 0, 5000]
    blocks = _check(ihip, 8, 2, lens, PLAN)
    for b, T in enumerate(lens):
        assert (blocks.view(len(lens), 2, -1)[b] >= 0).any() == (T > 320), (b, T)
    _check(ihip, 8, 2, lens, PLAN, "fp8-paged", True)


def test_pooled_over_all_heads(ihip):
    blocks = _check(ihip, 16, 4, [150000, 120000], PLAN, pooling=True)
    assert (blocks.view(2, 4, -1) == blocks.view(2, 4, -1)[:, :1]).all()


def test_cached_first_stage(ihip):
    """The last two stages recomputed from a list that an earlier query left, the sequences having grown since; both last lists land in
    the caller's state, and the same state without room for the scores taken together gives the same."""
    chunks, keeps = [s[0] for s in PLAN], [s[1] for s in PLAN]
    q, k, v, kw = _inputs(ihip, 8, 2, [150003, 99001], "bf16", False, 0)
    shape = torch.empty((2, 2, 150003, 0), dtype=torch.bfloat16)
    before = ihip.Layer(q, shape, torch.tensor([149990, 98700], dtype=torch.int32, device="cuda"), 1, 64, 256)
    L = ihip.Layer(q, shape, torch.tensor([150003, 99001], dtype=torch.int32, device="cuda"), 1, 64, 256)
    need = L.workspace_bytes(ihip.OP_DECODE_LAYER, chunks, keeps)
    got = []
    for size, launches in ((need, 1), (before.P * 4 * 2400 + 256 + L.workspace_bytes(ihip.OP_ATTN_DECODE, chunks[-1:], keeps[-1:]), 2)):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        state = before.mask_state(keeps)
        before.decode_layer_masked(-q, k, v, chunks, keeps, 0, state, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
        out = torch.empty((2, 8, 1, D), dtype=torch.bfloat16, device="cuda")
        assert _launches(ihip, lambda: L.decode_layer_masked(q, k, v, chunks, keeps, 1, state, ws=ws, out=out)) == launches
        got.append((state.cpu(), out.cpu().view(torch.int16)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("Hq,Hkv,stages,together", [
    (32, 8, ((64, 64), (16, 64), (4, 128)), False),       # a quarter kept, four heads: the searches read fewer rows than the pass
    (32, 8, ((64, 64), (16, 128), (4, 128)), True),
    (64, 8, ((64, 64), (16, 64), (4, 128)), True),        # eight heads: they read more
    (8, 8, ((64, 64), (16, 128), (4, 128)), False),       # one head
    (32, 8, ((32, 64), (16, 64), (4, 128)), False),       # parents of fewer than a wave's keys
    (32, 8, ((256, 256), (16, 2048), (4, 128)), False),   # more candidates than the selections take
])
def test_which_plans_go_together(ihip, Hq, Hkv, stages, together):
    q, k, v, kw = _inputs(ihip, Hq, Hkv, [140000], "bf16", False, 0)
    L = ihip.Layer(q, torch.empty((1, Hkv, 140000, 0), dtype=torch.bfloat16), torch.tensor([140000], dtype=torch.int32, device="cuda"), 1, 128, 1024)
    chunks, keeps = [s[0] for s in stages], [s[1] for s in stages]
    assert _launches(ihip, lambda: L.decode_layer(q, k, v, chunks, keeps)) == len(stages) - together


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("Hq", [8, 16])
def test_host_tier_rounds_alike(ihip, Hq, fp8):
    """K and V behind the host tier, N(0,1) data whose sums round: the bits of contiguous rows in device memory."""
    g = torch.Generator().manual_seed(Hq)
    T, chunks, keeps = 60000, [s[0] for s in PLAN], [s[1] for s in PLAN]
    q, k, v = torch.randn((1, Hq, 1, D), generator=g).bfloat16().cuda(), torch.randn((1, 2, T, D), generator=g), torch.randn((1, 2, T, D), generator=g)
    k, v = ((t.to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else t.bfloat16()) for t in (k, v))
    kw = {"kv_scales": (0.5, 0.25)} if fp8 else {}
    L = ihip.Layer(q, torch.empty((1, 2, T, 0), dtype=torch.bfloat16), torch.tensor([T], dtype=torch.int32, device="cuda"), 1, 64, 256)
    cache = ihip.HostKVCache(k.pin_memory(), v.pin_memory(), 64, 100, 50)
    try:
        lists = [torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda") for _ in range(2)]
        run = lambda *a, **b: L.decode_layer(q, *a, chunks, keeps, **kw, **b)  # noqa: E731
        want = [None]
        assert _launches(ihip, lambda: want.__setitem__(0, run(k.cuda(), v.cuda(), out_blocks=lists[0]))) == 2
        for _ in range(2):
            got = run(None, None, cache=cache, out_blocks=lists[1])
            cache.update()
            assert torch.equal(lists[0], lists[1]) and torch.equal(got.view(torch.int16), want[0].view(torch.int16))
    finally:
        cache.close()
