"""What bench.py counts as the bytes of a decode launch, for stages of their own and for stages scored together (CPU)."""
import bench

CHUNKS, KEEPS, SLOTS, ROWS, KEYS = [256, 64, 16, 4], [256, 256, 512, 1024], [4092, 1024, 1024, 2048], [36000.5, 7000, 4500, 7000], 1047424
NAMES = ["prune_decode.first.l256", "prune_decode.l64", "prune_decode.l16", "prune_decode.l4"]


def _bytes(ran):
    return bench.decode_kernel_bytes(CHUNKS, KEEPS, SLOTS, ROWS, KEYS, 256, ran)


def test_stages_of_their_own():
    for ran in ((), NAMES):
        assert _bytes(ran) == {
            "prune_decode.first.l256": 36000.5 * 256 + 4092 * 4, "select_blocks.first.l256": (4092 + 256) * 4,
            "prune_decode.l64": 7000 * 256 + 1024 * 4, "select_blocks.l64": (1024 + 256) * 4,
            "prune_decode.l16": 4500 * 256 + 1024 * 4, "select_blocks.l16": (1024 + 512) * 4,
            "prune_decode.l4": 7000 * 256 + 2048 * 4, "select_blocks.l4": (2048 + 1024) * 4}


def test_the_last_two_together():
    got = _bytes(NAMES[:3])
    assert got["prune_decode.l16"] == 1024 * 16 * 256 + (1024 + 4096) * 4
    assert got["select_blocks.l16"] == (1024 + 4096 + 512 + 1024) * 4
    assert got["prune_decode.l64"] == 7000 * 256 + 1024 * 4 and "prune_decode.l4" not in got


def test_all_in_one_pass():
    scores = 4092 * (1 + 4 + 16 + 64)
    assert _bytes(NAMES[:1]) == {"prune_decode.first.l256": KEYS * 256 + scores * 4, "select_blocks.first.l256": (scores + sum(KEEPS)) * 4}
