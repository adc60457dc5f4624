"""Decode attention alone (sparse_attn_decode.hip) against plain attention in float64: long splits and splits without a key, V near
both ends of what bf16 holds, and probabilities that have to go into the products whole."""
import math

import pytest
import torch

from test_gpu_decode_attn import _check, _turn

pytestmark = pytest.mark.gpu
D, HKV = 128, 2


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


def _over(ihip, q, k, v, n_stream, fmt, rope, unit, one_split):
    """One sequence, every token in the sink or the window.  -> |output - float64| less 2^-8 of it, at most, in units; the largest |V
    average| in units."""
    G, T, kw = q.shape[1] // HKV, k.shape[2], {}
    dev = lambda t: t.bfloat16().cuda()  # noqa: E731
    if fmt == "fp8":
        dev, kw["kv_scales"] = lambda t: t.to(torch.float8_e4m3fn).view(torch.uint8).cuda(), (1.0, 1.0)
    kk, qq, vv = k.double(), q.double(), v.bfloat16().double()
    if rope:
        ang = torch.arange(T, dtype=torch.float64).view(-1, 1) * 10000.0 ** (-2.0 * torch.arange(D // 2, dtype=torch.float64) / D)
        cos, sin = ang.cos().float(), ang.sin().float()
        kw["rope"] = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
        kk, qq = _turn(kk, torch.arange(T), cos, sin), _turn(qq, T - 1, cos, sin)
    if one_split:
        kw["ws"] = torch.empty(HKV * G * (D + 2) * 4, dtype=torch.uint8, device="cuda")
    L = ihip.Layer(q.bfloat16().cuda(), torch.empty((1, HKV, T, 0), dtype=torch.bfloat16), torch.tensor([T], dtype=torch.int32, device="cuda"),
                   1, T - n_stream, n_stream)
    out = L.sparse_attn_decode(q.bfloat16().cuda(), dev(k), dev(v), torch.empty((HKV, 0), dtype=torch.int32, device="cuda"), 4, **kw)
    out = (out[0] if isinstance(out, tuple) else out).cpu().double()[0, :, 0]
    want = torch.stack([torch.softmax(kk[0, h // G] @ qq[0, h, 0] / math.sqrt(D), 0) @ vv[0, h // G] for h in range(HKV * G)])
    return ((out - want).abs() - 2.0 ** -8 * want.abs()).max().item() / unit, want.abs().max().item() / unit


@pytest.mark.parametrize("fmt,rope", [("bf16", False), ("bf16", True), ("fp8", False), ("paged", False)])
@pytest.mark.parametrize("G", [1, 4])
def test_long_splits_and_splits_without_keys(ihip, G, fmt, rope):
    """128 problems of 8,857 slots, more than a GPU of 256 compute units takes at once in splits of 1,024: 1,120 slots and more to a split.
    Four fifths of the blocks are absent, so most splits hold no key at all."""
    _check(ihip, G, fmt, rope, [1700] * 2 + [303] * 61 + [9], 20, 37, 4, 2200, seed=G)


@pytest.mark.parametrize("rope", [False, True], ids=["plain", "streaming"])
@pytest.mark.parametrize("unit", [2.0 ** 122, 2.0 ** -118])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_large_and_small_v(ihip, G, unit, rope):
    """224 tokens, then 16 whose scores are 7.4 log2 units higher, in one split, so that a wave sees them after others: no
    probability may stand far above one, whatever the reference of the exponentials is, or its product with V overflows where
    neither the output (2^123) nor the sum (2^127) does.  Seen from the other end, a probability far below one must not push V's
    products out of the fp32 range.  Bound: fp32 sums of 240 products, 240 2^-24 of 2, and the output's own 2^-9."""
    g = torch.Generator().manual_seed(6)
    T = 240
    q, k = torch.zeros((1, HKV * G, 1, D)), torch.randn((1, HKV, T, D), generator=g).bfloat16().float()
    q[..., 126], k[..., 126] = 8, 7.25 * (torch.arange(T) >= T - 16).float()        # a dim that RoPE hardly turns
    v = torch.randn((1, HKV, T, D), generator=g).sign() * (1 + torch.rand((1, HKV, T, D), generator=g)) * unit
    over, _ = _over(ihip, q, k, v, 16, "bf16", rope, unit, True)
    assert over <= 2.0 ** -10, over


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
    T, a, b = 200, 21, 150
    q, k = torch.zeros((1, HKV * G, 1, D)), torch.zeros((1, HKV, T, D))
    at = 126 if rope else 0                           # the dims that RoPE turns least
    q[..., at], q[..., at + 1] = 1, 8
    for t, x in ((a, 1.0), (b, 0.9375)):
        k[:, :, t, at], k[:, :, t, at + 1] = x, 7
    v = torch.zeros((1, HKV, T, D))
    v[:, :, a] = (1 + 0.25 * torch.randint(0, 4, (HKV, D), generator=g).float()) * (1 - 2 * torch.randint(0, 2, (HKV, D), generator=g).float())
    v[:, :, b] = -v[:, :, a]
    over, largest = _over(ihip, q, k, v, 100, fmt, rope, 1.0, False)
    assert over <= 2.0 ** (-17 if rope else -20) * 1.75 and largest < 0.02, over
