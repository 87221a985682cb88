"""Sizes of the arena against what the kernels write into it (no GPU)."""
import pytest

import paper_1104_3830_amd as sk


@pytest.fixture
def tile_table():
    sk.lib()
    table = list(sk.loaded_tile_table)
    yield sk.set_tile_table
    sk.set_tile_table(table)


@pytest.mark.parametrize("n", [512, 1000, 2048, 4096])
@pytest.mark.parametrize("storage", [1, 2])
def test_stored_k_check_has_room_for_short_segments(tile_table, n, storage):
    """The FP64 check of a stored K writes n doubles per row segment of the
    column sweep, and a tuned table may make the segments 16 rows high: the
    arena grows by at least those of the added segments."""
    L = sk.lib()
    tile_table([(65536, 32)])
    tall = L.sk_arena_bytes(n, storage)
    tile_table([(65536, 16)])
    added = (n + 15) // 16 - (n + 31) // 32
    assert L.sk_arena_bytes(n, storage) - tall >= 8 * n * added
