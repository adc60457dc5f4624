"""The pass over the keys of kept chunks (prune_decode_nest.h with parents) with one and two heads a group, with chunks that the waves of a
workgroup share, and with absent parents of sequences of more than 2^30 keys, against the stage-by-stage kernels or lists known
from how the inputs are made; and the names that its kernels are timed under."""
import pytest
import torch

from test_gpu_tail import PLAN, _check, _inputs, _launches

pytestmark = pytest.mark.gpu
D = 128
MOST = ((64, 40), (16, 150), (4, 100))                # nearly all kept: with one and two heads the searches read fewer rows otherwise


@pytest.fixture(scope="module")
def ihip():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_08910_amd as pkg
    pkg.lib()
    return pkg


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "paged", "fp8-paged"])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("Hq", [2, 4])
def test_one_and_two_heads_a_group(ihip, Hq, fmt, rope):
    _check(ihip, Hq, 2, [150003, 99001], MOST, fmt, rope)


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "paged", "fp8-paged"])
@pytest.mark.parametrize("rope", [False, True], ids=["plain", "relative"])
@pytest.mark.parametrize("stages", [((256, 8), (128, 16), (4, 30)), ((512, 8), (256, 16), (8, 40))], ids=["128", "256"])
def test_chunks_of_more_than_a_wave(ihip, stages, rope, fmt):
    """Chunks of 128 and 256 keys, of which a wave scores 64: the waves of a workgroup meet in LDS.  The short sequences keep all of
    their first stage's chunks, the last one cut short by the end of the middle range, inside and at the end of a wave's keys."""
    _check(ihip, 16, 2, [150003, 64 + 256 + 256 * 7 + 133, 64 + 256 + 256 * 5 + 64, 64 + 256 + 3], stages, fmt, rope, seed=stages[0][0])


def test_kernels_are_named_by_the_stage_they_begin_with(ihip):
    q, k, v, kw = _inputs(ihip, 8, 2, [150003], "bf16", False, 0)
    L = ihip.Layer(q, torch.empty((1, 2, 150003, 0), dtype=torch.bfloat16), torch.tensor([150003], dtype=torch.int32, device="cuda"), 1, 64, 256)
    ihip.profile_read()
    ihip.profile_enable(True)
    try:
        L.decode_layer(q, k, v, [s[0] for s in PLAN], [s[1] for s in PLAN])
    finally:
        ihip.profile_enable(False)
    got = {name: n for name, (_, n) in ihip.profile_read().items()}
    assert got == {n: 1 for n in ("prune_decode.first.l64", "select_blocks.first.l64", "prune_decode.l16", "select_blocks.l16",
                                  "attn_decode_split", "attn_decode_merge")}


def test_absent_parents_of_very_long_sequences(ihip):
    """An absent parent (-1 in a cached first list) stands for no key, also where a sequence has more than 2^30 of them.  The
    tokens of a head share one row (stride 0), so the keys that an absent parent must not be taken for score as well as any."""
    T, chunks, keeps = (1 << 30) + (1 << 20), [s[0] for s in PLAN], [s[1] for s in PLAN]
    g = torch.Generator().manual_seed(1)
    q = torch.randint(-3, 4, (1, 8, 1, D), generator=g).bfloat16().cuda()
    k, v = (torch.randint(-3, 4, (1, 2, 1, D), generator=g).bfloat16().cuda().expand(1, 2, T, D) for _ in range(2))
    L = ihip.Layer(q, torch.empty((1, 2, T, 0), dtype=torch.bfloat16), torch.tensor([T], dtype=torch.int32, device="cuda"), 1, 64, 256)
    state = L.mask_state(keeps)
    first = torch.full((2, keeps[0]), -1, dtype=torch.int32)
    first[:, :10] = 64 + 64 * torch.arange(10) * (1 << 20)
    state[:2 * keeps[0]] = first.flatten().cuda()
    assert _launches(ihip, lambda: L.decode_layer_masked(q, k, v, chunks, keeps, 1, state)) == 1
    second, third = state[2 * keeps[0]:].cpu().split([2 * keeps[1], 2 * keeps[2]])
    want = (first[:, :10, None] + 16 * torch.arange(4)).flatten(1)
    assert torch.equal(second.view(2, -1)[:, :40], want) and (second.view(2, -1)[:, 40:] == -1).all()
    want = (want[:, :, None] + 4 * torch.arange(4)).flatten(1)[:, :100]
    assert torch.equal(third.view(2, -1), want)
