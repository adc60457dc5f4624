"""Prefill attention whose key lists are cut into splits (few problems) against the oracle and against the same call without
scratch, which takes one split.  Bounds: 1e-2 to 2e-2 against the oracle as in the other prefill tests; between the two ways the
probabilities are rounded to bf16 (2^-9) relative to different references, and the outputs once more: 2^-7 of the largest
output; log-sum-exp of fp32 sums in another order: 2e-5."""
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


def close(a, b):
    assert (a.float() - b.float()).abs().max() <= 2.0 ** -7 * a.float().abs().max()


@pytest.mark.parametrize("variant", ["bf16", "paged", "rope", "fp8", "rope-fp8"])
@pytest.mark.parametrize("b_q,Hq,Hkv,Tq,n_blocks", [
    (64, 8, 2, 128, 100),      # eight waves
    (64, 16, 2, 64, 61),       # eight heads: two workgroups of four heads to a problem
    (32, 8, 2, 96, 100), (64, 2, 2, 128, 77), (32, 1, 1, 32, 200),
    (16, 8, 2, 48, 90),        # the 16x16 kernel
], ids=["q64", "q64-8heads", "q32", "q64-1head", "one-wave", "q16"])
def test_splits_against_oracle_and_one_split(ihip, orc, b_q, Hq, Hkv, Tq, n_blocks, variant):
    """Two sequences, the second so short that its later splits hold no key (or only masked ones), lists with empty slots."""
    block, n_stream = 16, 256
    w = configs.shrink(configs.CFG4, B=2, Hq=Hq, Hkv=Hkv, T=6000 + Tq, Tq=Tq, b_q=b_q, n_stream=n_stream, stages=((block, n_blocks),))
    q, k, v, sl, _ = configs.make_inputs(w, 3)
    lens = [w.T, Tq + 40]
    sl = torch.tensor(lens, dtype=torch.int32)
    starts = torch.full((w.B * Hkv * w.Mq, n_blocks), -1, dtype=torch.int32)
    n_mid = (w.T - Tq - w.n_sink - n_stream) // block
    for p in range(Hkv * w.Mq):                  # sequence 0 only: the other's middle range is empty
        pick = gen.distinct_ints(6, 100 + p, n_blocks, n_mid).sort().values[:n_blocks - p % 3]
        starts[p, :len(pick)] = (w.n_sink + pick * block).to(torch.int32)
    cos, sin = gen.rope_table(4096, w.d)
    spec = orc.RopeSpec(cos.numpy(), sin.numpy(), attn="streaming") if "rope" in variant else None
    kw, ok, ov = {}, k, v
    kd, vd = k.cuda(), v.cuda()
    if "rope" in variant:
        kw["rope"] = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_NONE, ihip.ROPE_STREAMING)
    if "fp8" in variant:
        s = 1 / 64
        k8, v8 = gen.to_e4m3(k, s), gen.to_e4m3(v, s)
        kw["kv_scales"] = (s, s)
        kd, vd = k8.cuda(), v8.cuda()
        ok, ov = ((t.view(torch.float8_e4m3fn).float() * s).bfloat16() for t in (k8, v8))      # exact: a power of two
    if variant == "paged":
        page, n = 32, -(-w.T // 32)
        order = torch.randperm(2 * n, generator=torch.Generator().manual_seed(5))
        pools = []
        for t in (k, v):
            full = torch.zeros((2, Hkv, n * page, w.d), dtype=t.dtype)
            full[:, :, :w.T] = t
            pool = torch.empty((2 * n, Hkv, page, w.d), dtype=t.dtype)
            pool[order] = full.view(2, Hkv, n, page, w.d).permute(0, 2, 1, 3, 4).reshape(2 * n, Hkv, page, w.d)
            pools.append(pool.cuda())
        kw["paged"] = ihip.PagedKV(pools[0], pools[1], order.to(torch.int32).view(2, n).contiguous().cuda())
    L = ihip.Layer(q.cuda(), kd, sl.cuda(), b_q, w.n_sink, n_stream)
    need = L.workspace_bytes(ihip.OP_ATTN_PREFILL, [block], [n_blocks])
    assert need > 1 << 16                        # the call is split
    got = []
    for size in (need, 256):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        out, lse = L.sparse_attn_prefill(q.cuda(), kd, vd, starts.cuda(), block, want_lse=True, ws=ws, **kw)
        torch.cuda.synchronize()
        got.append((out.cpu(), lse.cpu()))
        assert bool((ws == 0xA5).all()) == (size == 256)
    close(got[1][0], got[0][0])
    np.testing.assert_allclose(got[0][1].numpy(), got[1][1].numpy(), rtol=2e-5, atol=2e-5)
    o = orc.Oracle(q, ok, ov, lens, b_q, w.n_sink, n_stream, rope=spec)
    for b, g, m in ((0, 0, 0), (0, Hkv - 1, w.Mq - 1), (1, 0, w.Mq - 1)):
        s = starts[(b * Hkv + g) * w.Mq + m]
        s = s[s >= 0].numpy()
        ref, ref_lse = o.attend(b, g, m, s, np.full(len(s), block, np.int32))
        rows = slice(m * b_q, (m + 1) * b_q)
        assert np.abs(got[0][0][b, g * w.G:(g + 1) * w.G, rows].float().numpy() - ref).max() <= (1e-2 if spec is None else 2e-2), (b, g, m)


@pytest.mark.parametrize("b_q", [64, 32, 16])
def test_layer_with_and_without_room_for_splits(ihip, b_q):
    """E4M3 pages with RoPE through the layer call: same lists (the pruning does not change), outputs as close as above."""
    Tq, Hq, Hkv, page, T = 2 * b_q, 8, 2, 16, 4000
    g = torch.Generator().manual_seed(1)
    q = torch.randn((1, Hq, Tq, 128), generator=g).bfloat16().cuda()
    n = -(-T // page)
    k, v = (torch.randn((n, Hkv, page, 128), generator=g).mul(64).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8).cuda() for _ in range(2))
    pg = ihip.PagedKV(k, v, torch.randperm(n, generator=g).to(torch.int32).view(1, n).contiguous().cuda())
    cos, sin = gen.rope_table(4096, 128)
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_RELATIVE, ihip.ROPE_STREAMING)
    L = ihip.Layer(q, torch.empty((1, Hkv, T, 0), dtype=torch.bfloat16), torch.tensor([T], dtype=torch.int32, device="cuda"), b_q, 64, 512)
    chunks, keeps = [32, 8], [60, 200]
    need = L.workspace_bytes(ihip.OP_PREFILL_LAYER, chunks, keeps)
    got = []
    for size in (need, need - L.workspace_bytes(ihip.OP_ATTN_PREFILL, chunks[-1:], keeps[-1:])):       # ... and no scratch for the attention
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
        out = L.prefill_layer(q, None, None, chunks, keeps, ws=ws, rope=rp, paged=pg, kv_scales=(1 / 64, 1 / 64), out_blocks=blocks)
        torch.cuda.synchronize()
        got.append((out.cpu(), blocks.cpu()))
    assert torch.equal(got[0][1], got[1][1])
    close(got[1][0], got[0][0])
    assert not torch.equal(got[0][0], got[1][0])             # two ways
