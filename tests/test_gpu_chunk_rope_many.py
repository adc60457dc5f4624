"""Chunk-indexed RoPE prefill pruning in launches of many workgroups (three to a compute unit with 64-query blocks and four heads)
against the same query blocks one by one (few workgroups, which the oracle tests hold): the same arithmetic, so the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from workloads import gen  # noqa: E402


@pytest.mark.parametrize("b_q,Hq,Hkv", [(64, 32, 8), (64, 64, 8), (32, 32, 8), (16, 32, 8), (64, 16, 8), (16, 64, 8)],
                         ids=["q64", "q64-8heads", "q32", "q16", "q64-2heads", "q16-8heads"])
def test_many_workgroups_against_few(b_q, Hq, Hkv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as ihip
    nb, l, n_sink, n_stream = 8, 64, 100, 512
    T = 33001
    g = torch.Generator().manual_seed(b_q)
    q = torch.randn((1, Hq, nb * b_q, 128), generator=g).bfloat16().cuda()
    k = torch.randn((1, Hkv, T, 128), generator=g).bfloat16().cuda()
    cos, sin = gen.rope_table(2048, 128)
    rp = ihip.Rope(cos.cuda(), sin.cuda(), ihip.ROPE_CHUNK_INDEXED, ihip.ROPE_NONE)
    L = ihip.Layer(q, k, torch.tensor([T], dtype=torch.int32, device="cuda"), b_q, n_sink, n_stream)
    many, rep = L.prune_stage(q, k, l, rope=rp, want_rep=True)
    for m in (0, nb - 1):
        one = q[:, :, m * b_q:(m + 1) * b_q].contiguous()
        seq = T - (nb - 1 - m) * b_q
        L1 = ihip.Layer(one, k, torch.tensor([seq], dtype=torch.int32, device="cuda"), b_q, n_sink, n_stream)
        few, rep1 = L1.prune_stage(one, k, l, rope=rp, want_rep=True)
        n = (seq - n_stream - n_sink + l - 1) // l
        assert torch.isfinite(few[:, :n]).all()
        assert torch.equal(many.view(Hkv, nb, -1)[:, m, :n], few[:, :n])
        assert torch.equal(rep[0, :, m, :n], rep1[0, :, 0, :n])
