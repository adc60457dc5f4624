"""Decode stages that are large enough for the matrix-core search (prune_decode_tile.h) by the lines of decode_on_tiles, against the
same sequences one at a time, which stay on the vector kernels: forms that no other test brings above its line.  E4M3 rows with
one and two heads a group, contiguous and in pages, with and without RoPE; chunks of one and two keys with four and eight heads.
Inputs are whole numbers (and quarter turns), so every score is exact in both kernels and the lists have to be the same, ties
included.  The batch's slots are no multiple of a workgroup's chunks."""
import pytest
import torch

pytestmark = pytest.mark.gpu
D, HKV, SINK, STREAM = 128, 8, 64, 128


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


def _whole(shape, fp8, g):
    t = torch.randint(-2, 3, shape, generator=g, device="cuda", dtype=torch.int8)
    if not fp8:
        return t.bfloat16()
    return torch.tensor([0xC0, 0xB8, 0x00, 0x38, 0x40], dtype=torch.uint8, device="cuda")[(t + 2).long()]      # E4M3 of -2 .. 2


def _lists(ihip, q, kv, table, lens, chunk, keep, kw, parents=None):
    """The kept lists of one stage: a first one, or (parents: starts of chunks of 4 * chunk keys) a later one."""
    T = max(lens)
    L = ihip.Layer(q, torch.empty((len(lens), HKV, T, 0), dtype=torch.bfloat16), torch.tensor(lens, dtype=torch.int32, device="cuda"), 1, SINK, STREAM)
    kw = dict(kw)
    if table is not None:
        kw["paged"] = ihip.PagedKV(kv, kv, table)
    chunks, keeps = ([chunk], [keep]) if parents is None else ([4 * chunk, chunk], [parents.shape[1], keep])
    state = L.mask_state(keeps)
    if parents is not None:
        state[:parents.numel()] = parents.flatten()
    ihip.profile_read()
    ihip.profile_enable(True)
    try:
        L.decode_layer(q, kv, kv, chunks, keeps, stage_starts=state, stage_due=[0, 1][2 - len(chunks):] if parents is not None else [1], **kw)
    finally:
        ihip.profile_enable(False)
    names = [n for n in ihip.profile_read() if n.startswith("prune")]
    assert names == ["prune_decode%s.l%d" % (".first" if parents is None else "", chunk)], names
    return state[-L.P * keep:].view(L.P, keep).cpu()


def _check(ihip, G, fmt, rope, chunk, per_cu, later):
    """per_cu: workgroups of the matrix-core kernel a compute unit to be reached, of 4 waves with 64 / G chunks each (chunks of
    four: 16 to a wave)."""
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    per_wg = 4 * (16 if chunk == 4 else 64 // G)
    B = 8
    wgs = -(-int(per_cu * cu) // (B * HKV)) + 1                 # of a problem
    slots = (wgs - 1) * per_wg + per_wg // 3                    # the last one is a third full
    keys = slots * chunk
    T = SINK + STREAM + keys - chunk // 2                       # the last chunk is cut short
    lens = [T] + [T - chunk * (7 * b + 1) - b for b in range(1, B)]
    g = torch.Generator(device="cuda").manual_seed(chunk * 10 + G)
    fp8, kw, table = "fp8" in fmt, {}, None
    if "paged" in fmt:
        n = -(-T // 16)
        table = torch.randperm(B * n, generator=g, device="cuda").to(torch.int32).view(B, n).contiguous()
        kv = _whole((B * n, HKV, 16, D), fp8, g)
    else:
        kv = _whole((B, HKV, T, D), fp8, g)
    if fp8:
        kw["kv_scales"] = (1.0, 1.0)
    q = torch.randint(-3, 4, (B, HKV * G, 1, D), generator=g, device="cuda").bfloat16()
    keep = 300
    if rope:
        turn = torch.arange(SINK + STREAM + keep * chunk + 8, device="cuda") % 4
        c = torch.tensor([1.0, 0.0, -1.0, 0.0], device="cuda")[turn].view(-1, 1).repeat(1, D // 2).contiguous()
        s = torch.tensor([0.0, 1.0, 0.0, -1.0], device="cuda")[turn].view(-1, 1).repeat(1, D // 2).contiguous()
        kw["rope"] = ihip.Rope(c, s, ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    parents = None
    if later:                                                   # the chunks of four children, up to four of them left out
        n = -(-slots // 4)
        parents = torch.full((B * HKV, n), -1, dtype=torch.int32, device="cuda")
        for p in range(B * HKV):
            mid = lens[p // HKV] - SINK - STREAM
            at = torch.randperm(-(-mid // (4 * chunk)), generator=g, device="cuda")[:n - (p % 5)].sort().values
            parents[p, :len(at)] = (SINK + at * 4 * chunk).to(torch.int32)
    got = _lists(ihip, q, kv, table, lens, chunk, keep, kw, parents).view(B, HKV, keep)
    for b in range(B):
        kvb, tb = (kv, table[b:b + 1]) if table is not None else (kv[b:b + 1, :, :lens[b]], None)
        pb = parents.view(B, HKV, -1)[b].contiguous() if later else None
        assert torch.equal(got[b], _lists(ihip, q[b:b + 1].contiguous(), kvb, tb, lens[b:b + 1], chunk, keep, kw, pb)), b


@pytest.mark.parametrize("later", [False, True], ids=["first", "later"])
@pytest.mark.parametrize("chunk,per_cu", [(4, 2), (16, 3), (64, 3)])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("fmt", ["fp8", "fp8-paged"])
@pytest.mark.parametrize("G", [1, 2])
def test_few_heads_over_e4m3(ihip, G, fmt, rope, chunk, per_cu, later):
    _check(ihip, G, fmt, rope, chunk, per_cu, later)


@pytest.mark.parametrize("chunk", [1, 2])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("fmt", ["bf16", "paged", "fp8", "fp8-paged"])
@pytest.mark.parametrize("G", [4, 8])
def test_chunks_of_one_and_two_keys(ihip, G, fmt, rope, chunk):
    _check(ihip, G, fmt, rope, chunk, 4, True)
