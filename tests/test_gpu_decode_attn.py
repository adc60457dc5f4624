"""Decode attention alone (sparse_attn_decode.hip) against plain attention in float64, where its tiles of 16 slots, four-token row
groups and splits end: lists that fill no tile, one tile, one wave more than a tile, several splits; blocks cut short at the end
of the middle range, absent blocks, a sink longer than the sequence; scores that outgrow the reference of the exponentials; and V
near both ends of what bf16 holds.

Bounds.  Scores and sums are fp32 and the probabilities go into the products whole (24 bits; test_probabilities_are_whole): an output is the fp32 result
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


def _check(ihip, G, fmt, rope, lens, n_sink, n_stream, block, n_blocks, grow=0.0, seed=0, v_unit=1.0, step=False, only=None):
    g = torch.Generator().manual_seed(seed)
    Hkv, B, T = 2, len(lens), max(lens)
    Hq = Hkv * G
    q = torch.randn((B, Hq, 1, D), generator=g).bfloat16()
    k, v = (torch.randn((B, Hkv, T, D), generator=g) for _ in range(2))
    if grow:                                          # keys along the first head, longer and longer: scores climb with the position
        k = k + q[:, ::G, 0].float().unsqueeze(2) * torch.linspace(-grow, grow, T).view(1, 1, T, 1)
    if step:                                          # the window 8 * 7.25 / sqrt(128) higher, in a dim that RoPE hardly turns
        q, k[..., 126] = torch.zeros_like(q), 7.25 * (torch.arange(T) >= T - n_stream).float()
        q[..., 126] = 8
        v = v.sign() * (1 + torch.rand(v.shape, generator=g))
    v = v * v_unit                                    # a power of two
    kw = {"ws": torch.empty(B * Hq * (D + 2) * 4, dtype=torch.uint8, device="cuda")} if step else {}        # one coarse split
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
    for b in range(B) if only is None else only:
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
            bound = 2.0 ** -8 * want.abs() + 2.0 ** -10 * v_unit
            over = ((out[b, h, 0] - want).abs() - bound).max().item()
            assert over <= 0, (b, h, over)
            assert abs(lse[b, h, 0] - r) <= 1e-5 * max(1.0, r.abs().item()), (b, h, lse[b, h, 0], r)


# RoPE over pages and E4M3 rows has entry points through the layer only (test_gpu_combos.py)
FORMS = pytest.mark.parametrize("fmt,rope", [("bf16", False), ("bf16", True), ("fp8", False), ("paged", False)])


@FORMS
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_groups_and_storage(ihip, G, fmt, rope):
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


@FORMS
@pytest.mark.parametrize("G", [1, 4])
def test_long_splits_and_splits_without_keys(ihip, G, fmt, rope):
    """128 problems of 8,857 slots, more than a GPU of 256 compute units takes at once in splits of 1,024: 1,120 slots and more to a split.
    Four fifths of the blocks are absent, so most splits hold no key at all."""
    _check(ihip, G, fmt, rope, [1700] * 62 + [9, 0], 20, 37, 4, 2200, seed=G, only=(0, 30, 61, 62))


@pytest.mark.parametrize("G", [1, 4, 8])
def test_scores_that_outgrow_the_reference(ihip, G):
    """Scores climb from about -100 to 100 along the list: the reference moves in nearly every tile."""
    _check(ihip, G, "bf16", False, [1500], 16, 64, 4, 300, grow=8.0, seed=3)
    _check(ihip, G, "fp8", False, [1500], 16, 64, 4, 300, grow=8.0, seed=4)
    _check(ihip, G, "bf16", True, [1500], 16, 64, 4, 300, grow=8.0, seed=5)


@pytest.mark.parametrize("rope", [False, True], ids=["plain", "streaming"])
@pytest.mark.parametrize("unit", [2.0 ** 122, 2.0 ** -118])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_large_and_small_v(ihip, G, unit, rope):
    """224 tokens, then 16 whose scores are 7.4 log2 units higher, in one split, so that a wave sees them after others: no
    probability may stand far above one, whatever the reference of the exponentials is, or its product with V overflows where
    neither the output (2^123) nor the sum (2^127) does.  Seen from the other end, a probability far below one must not push V's
    products out of the fp32 range."""
    _check(ihip, G, "bf16", rope, [240], 64, 16, 4, 40, seed=6, v_unit=unit, step=True)


@pytest.mark.parametrize("fmt,rope", [("bf16", False), ("bf16", True), ("fp8", False)])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_probabilities_are_whole(ihip, G, fmt, rope):
    """Two tokens hold nearly all of the softmax, in nearly equal parts, and their V rows are each other's negatives: the output is
    some 0.002 of |V|, the difference of two probabilities.  Probabilities of a single bf16 part (2^-9) would be off by a quarter of
    it, sixty times the bound; a third part beyond the second (2^-17) is more than a bf16 output can show.  The dot products are
    exact, a score in log2 units (about 7.3) is rounded to 2^-22, its distance to the reference (at most 8) to 2^-22 and the
    exponential to 2^-23: 2^-20.7 of V at most, and the output's own 2^-9.  With RoPE the products of turned dims add up to 57,
    whose 128 roundings are the larger part: 2^-17."""
    g = torch.Generator().manual_seed(G)
    Hkv, T, a, b = 2, 200, 21, 150
    q, k = torch.zeros((1, Hkv * G, 1, D)), torch.zeros((1, Hkv, T, D))
    at = 126 if rope else 0                           # the dims that RoPE turns least
    q[..., at], q[..., at + 1] = 1, 8
    for t, x in ((a, 1.0), (b, 0.9375)):
        k[:, :, t, at], k[:, :, t, at + 1] = x, 7
    v = torch.zeros((1, Hkv, T, D))
    v[:, :, a] = (1 + 0.25 * torch.randint(0, 4, (Hkv, D), generator=g).float()) * (1 - 2 * torch.randint(0, 2, (Hkv, D), generator=g).float())
    v[:, :, b] = -v[:, :, a]
    kw = {}
    dev = lambda t: t.bfloat16().cuda()  # noqa: E731
    if fmt == "fp8":
        dev, kw["kv_scales"] = lambda t: t.to(torch.float8_e4m3fn).view(torch.uint8).cuda(), (1.0, 1.0)
    kk, qq = k.double(), q.double()
    if rope:
        ang = torch.arange(T, dtype=torch.float64).view(-1, 1) * 10000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64) / D)
        cos, sin = ang.cos().float(), ang.sin().float()
        kw["rope"] = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
        kk, qq = _turn(kk, torch.arange(T), cos, sin), _turn(qq, T - 1, cos, sin)
    L = ihip.Layer(dev(q) if fmt != "fp8" else q.bfloat16().cuda(), torch.empty((1, Hkv, T, 0), dtype=torch.bfloat16),
                   torch.tensor([T], dtype=torch.int32, device="cuda"), 1, 100, 100)
    out = L.sparse_attn_decode(q.bfloat16().cuda(), dev(k), dev(v), torch.empty((Hkv, 0), dtype=torch.int32, device="cuda"), 4, **kw)
    out = (out[0] if isinstance(out, tuple) else out).cpu().double()[0, :, 0]
    for h in range(Hkv * G):
        want = torch.softmax(kk[0, h // G] @ qq[0, h, 0] / math.sqrt(D), 0) @ v[0, h // G].double()
        over = ((out[h] - want).abs() - 2.0 ** -8 * want.abs()).max().item()
        assert over <= 2.0 ** (-17 if rope else -20) * 1.75 and want.abs().max() < 0.02, (h, over)
