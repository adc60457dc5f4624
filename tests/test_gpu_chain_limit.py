"""The one-launch selections (select_chain.hip) where the bin of the K-th best score holds exactly as many candidates as a wave has lanes,
or one more: nothing else scores within 64 of the tied ones, many times a bin's width (1.5 / 512 of the range, 2,400 at most).  Scores are
whole numbers, exact in every kernel; the lists are compared with the ones known from how the inputs are made, and the
launches are counted."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pooling", [False, True], ids=["kv-head", "all-heads"])
@pytest.mark.parametrize("n_slots", [400, 1500])
@pytest.mark.parametrize("ties", [1, 2, 63, 64, 65, 300])
def test_equal_scores_alone_in_their_bin(ties, n_slots, pooling):
    import paper_2502_08910_amd as ihip
    n_sink, n_stream, Hkv, D = 64, 256, 2, 128
    T = n_sink + n_stream + 8 * n_slots
    g = torch.Generator().manual_seed(ties)
    above = (n_slots - ties) // 2
    rank = torch.randperm(n_slots, generator=g)           # of the slots: the first `above` are better than the tied ones, the rest worse
    value = torch.where(rank < above, 2064 + rank, torch.where(rank < above + ties, torch.tensor(2000), 1936 - rank))
    q = torch.zeros((1, 2 * Hkv, 1, D))
    q[..., 0], q[..., 1] = 64, 1                          # score = 64 * k0 + k1
    k = torch.zeros((1, Hkv, T, D))
    v = value.repeat_interleave(8)
    k[:, :, n_sink:T - n_stream, 0], k[:, :, n_sink:T - n_stream, 1] = (v // 64).float(), (v % 64).float()
    q, k = q.bfloat16().cuda(), k.bfloat16().cuda()
    keep = above + (ties + 1) // 2
    chunks, keeps = [8, 4], [keep, 2 * keep]
    L = ihip.Layer(q, k, torch.tensor([T], dtype=torch.int32, device="cuda"), 1, n_sink, n_stream)
    blocks = torch.empty((L.P, keeps[-1]), dtype=torch.int32, device="cuda")
    kw = {"pooling": ihip.binding.POOL_ALL_HEADS} if pooling else {}
    ihip.profile_read()
    ihip.profile_enable(True)
    try:
        L.decode_layer(q, k, k, chunks, keeps, out_blocks=blocks, **kw)
    finally:
        ihip.profile_enable(False)
    launches = {name: n for name, (_, n) in ihip.profile_read().items() if not name.startswith("attn")}
    assert launches == {"prune_decode.first.l8": 1, "select_blocks.first.l8": 1}, launches
    best = torch.sort(value, descending=True, stable=True).indices[:keep].sort().values
    want = (n_sink + best.view(-1, 1) * 8 + torch.tensor([0, 4])).flatten().to(torch.int32)
    assert torch.equal(blocks.cpu(), want.expand(Hkv, -1))
