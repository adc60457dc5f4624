"""Decode attention alone (sparse_attn_decode.hip) against plain attention in float64, where its tiles of 16 slots, four-token row
groups and splits end: lists that fill no tile, one tile, one wave more than a tile, several splits; blocks cut short at the end
of the middle range, absent blocks, a sink longer than the sequence; and scores that outgrow the reference of the exponentials.

Bounds.  Scores and sums are fp32 and the probabilities go into the products whole (24 bits): an output is the fp32 result
rounded to bf16, half a unit in the last of 8 bits <= 2^-8 of it, and fp32 sums of n products add up to about n 2^-24 of the
largest |V| (n < 4096: 2^-12 of 4).  With RoPE the turned dims are fp32 too."""
import math

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


def _turn(x, pos, cos, sin):
    c, s = cos[pos].double(), sin[pos].double()
    e, o = x[..., 0::2], x[..., 1::2]
    return torch.stack((e * c - o * s, e * s + o * c), dim=-1).flatten(-2)


def _check(ihip, G, fmt, rope, lens, n_sink, n_stream, block, n_blocks, grow=0.0, seed=0):
    g = torch.Generator().manual_seed(seed)
    Hkv, B, T = 2, len(lens), max(lens)
    Hq = Hkv * G
    q = torch.randn((B, Hq, 1, D), generator=g).bfloat16()
    k, v = (torch.randn((B, Hkv, T, D), generator=g) for _ in range(2))
    if grow:                                          # keys along the first head, longer and longer: scores climb with the position
        k = k + q[:, ::G, 0].float().unsqueeze(2) * torch.linspace(-grow, grow, T).view(1, 1, T, 1)
    kw = {}
    if fmt == "fp8":
        k, v = (t.clamp(-448, 448).to(torch.float8_e4m3fn) for t in (k, v))
        kw["kv_scales"] = (1.0, 1.0)
    else:
        k, v = k.bfloat16(), v.bfloat16()
    lens_t = torch.tensor(lens, dtype=torch.int32)
    # distinct blocks of the middle range, ascending, -1 padded; the last one is kept wherever there are any, cut short or not
    starts = torch.full((B * Hkv, n_blocks), -1, dtype=torch.int32)
    for p in range(B * Hkv):
        n = max(0, -(-(lens[p // Hkv] - n_stream - n_sink) // block))
        take = torch.randperm(n, generator=g)[:max(0, n_blocks - (p & 1))]
        if len(take):
            take[0] = n - 1
        take = take.unique().to(torch.int32)
        starts[p, :len(take)] = n_sink + take * block
    dev = lambda t: t.view(torch.uint8).cuda() if t.dtype == torch.float8_e4m3fn else t.cuda()  # noqa: E731
    kd, vd = dev(k), dev(v)
    L = ihip.Layer(q.cuda(), torch.empty((B, Hkv, T, 0), dtype=torch.bfloat16), lens_t.cuda(), 1, n_sink, n_stream)
    if rope:
        j = torch.arange(D // 2, dtype=torch.float64)
        ang = torch.arange(n_sink + n_blocks * block + n_stream, dtype=torch.float64).view(-1, 1) * 10000.0 ** (-2.0 * j / D)
        cos, sin = ang.cos().float(), ang.sin().float()
        kw["rope"] = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
    if fmt == "paged":
        page, n = 16, -(-T // 16)
        order = torch.randperm(B * n, generator=g)
        pools = []
        for t in (k, v):
            full = torch.zeros((B, Hkv, n * page, D), dtype=t.dtype)
            full[:, :, :T] = t
            pool = torch.empty((B * n, Hkv, page, D), dtype=t.dtype)
            pool[order] = full.view(B, Hkv, n, page, D).permute(0, 2, 1, 3, 4).reshape(B * n, Hkv, page, D)
            pools.append(pool.cuda())
        kw["paged"] = ihip.PagedKV(pools[0], pools[1], order.to(torch.int32).view(B, n).contiguous().cuda())
    out, lse = L.sparse_attn_decode(q.cuda(), kd, vd, starts.cuda(), block, want_lse=True, **kw)
    out, lse = out.cpu().double(), lse.cpu().double()
    for b in range(B):
        E = lens[b]
        hi = E - n_stream
        for h in range(Hq):
            kept = starts[b * Hkv + h // G].long()
            mid = (kept[kept >= 0].view(-1, 1) + torch.arange(block)).flatten()
            pos = torch.cat([torch.arange(min(n_sink, E)), mid[mid < hi], torch.arange(max(hi, n_sink), max(E, n_sink))])
            kk, qq = k[b, h // G, pos].double(), q[b, h, 0].double()
            if rope:
                kk, qq = _turn(kk, torch.arange(len(pos)), cos, sin), _turn(qq, len(pos) - 1, cos, sin)
            s = kk @ qq / math.sqrt(D)
            r = torch.logsumexp(s, 0)
            want = (s - r).exp() @ v[b, h // G, pos].double()
            bound = 2.0 ** -8 * want.abs() + 2.0 ** -10
            over = ((out[b, h, 0] - want).abs() - bound).max().item()
            assert over <= 0, (b, h, over)
            assert abs(lse[b, h, 0] - r) <= 1e-5 * max(1.0, r.abs().item()), (b, h, lse[b, h, 0], r)


@pytest.mark.parametrize("rope", [False, True], ids=["plain", "streaming"])
@pytest.mark.parametrize("fmt", ["bf16", "fp8", "paged"])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_groups_and_storage(ihip, G, fmt, rope):
    if fmt != "bf16" and rope:
        pytest.skip("RoPE over pages and E4M3 rows has entry points through the layer only (test_gpu_combos.py)")
    _check(ihip, G, fmt, rope, [701, 303], 20, 37, 4, 21, seed=G)


@pytest.mark.parametrize("lens,n_sink,n_stream,block,n_blocks", [
    ([40], 3, 5, 1, 3),                    # less than a tile
    ([90], 8, 8, 4, 0),                    # a tile, no blocks
    ([90], 8, 8, 4, 1),                    # a tile and four slots
    ([200, 90], 31, 29, 8, 1),             # one slot over four tiles: a second round of one wave
    ([3000, 9, 60], 64, 100, 16, 101),     # several splits; sequences shorter than the sink and than sink and window
    ([5000], 128, 1024, 4, 900),           # splits of many tiles
], ids=lambda x: str(x) if isinstance(x, list) else None)
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "streaming"])
def test_ends_of_tiles_and_splits(ihip, lens, n_sink, n_stream, block, n_blocks, rope):
    _check(ihip, 4, "bf16", rope, lens, n_sink, n_stream, block, n_blocks, seed=len(lens))


@pytest.mark.parametrize("G", [1, 4, 8])
def test_scores_that_outgrow_the_reference(ihip, G):
    """Scores climb from about -100 to 100 along the list: the reference moves in nearly every tile."""
    _check(ihip, G, "bf16", False, [1500], 16, 64, 4, 300, grow=8.0, seed=3)
    _check(ihip, G, "fp8", False, [1500], 16, 64, 4, 300, grow=8.0, seed=4)
    _check(ihip, G, "bf16", True, [1500], 16, 64, 4, 300, grow=8.0, seed=5)
