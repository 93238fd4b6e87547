"""The planner's choice of the row tile: by the ranges of a compute-heavy step, by shared key ranges of one bound by
HBM (no GPU: the work list is a host function)."""
import numpy as np
import pytest

from paper_2505_21889_amd import binding as E


def tile_of(cached, new, heads, d):
    pages = -(-(np.array(cached) + np.array(new)) // 16)
    table = np.zeros((len(cached), int(pages.max())), np.int32)
    desc = E.BatchDesc(cached, new, table, heads[0], heads[1], d, 16, 1 << 24)
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 512)
    try:
        items = E.efim_extend_plan_items(desc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
    return int(items["row_count"].max())


@pytest.mark.parametrize("d,keys,tile", [(128, 1900, 128), (128, 2200, 256), (64, 3900, 128), (64, 4300, 256)])
def test_compute_heavy_steps_by_their_ranges(d, keys, tile):
    assert tile_of([keys - 128] * 16, [256] * 16, (32, 8), d) == tile


@pytest.mark.parametrize("new,tile", [([300] * 40, 128), ([150] * 40, 150)])
def test_steps_bound_by_hbm_by_their_shared_ranges(new, tile):
    """32/32 heads: 300 rows per head are two tiles of 256 and read the keys twice; 150 are one."""
    assert tile_of([2000] * len(new), new, (32, 32), 128) == tile


def test_a_step_that_the_static_call_takes_in_256_rows_stays_within_its_limits():
    """Work list (48 bytes per item) of at most 2 MiB and partial results of at most 30 MiB wherever 256 rows stay there;
    where they do not either, the tile that the ranges ask for."""
    rng = np.random.default_rng(5)
    list_too_long = ([100] * 900, [200] * 900, (32, 8), 128)   # 28800 items of 256 rows (1.4 MB), 50400 of 128 (2.4 MB)
    both_too_long = ([100] * 2000, [200] * 2000, (32, 8), 128) # 64000 and 112000
    cases = []
    for _ in range(40):
        batch = int(rng.integers(1, 24))
        heads = [(32, 8), (28, 4), (32, 32)][int(rng.integers(0, 3))]
        cases.append((rng.integers(64, 3000, batch).tolist(), rng.integers(1, 600, batch).tolist(), heads, 128))

    def sizes(row_tile, case):
        cached, new, heads, d = case
        pages = -(-(np.array(cached) + np.array(new)) // 16)
        table = np.zeros((len(cached), int(pages.max())), np.int32)
        desc = E.BatchDesc(cached, new, table, heads[0], heads[1], d, 16, 1 << 24)
        E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 512)
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
        try:
            return len(E.efim_extend_plan_items(desc)) * 48, E.efim_extend_workspace_bytes(desc)
        finally:
            E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
            E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)

    limits = (2 << 20, 30 << 20)
    for case, tile in ((list_too_long, 256), (both_too_long, 128)):
        narrow, wide = sizes(128, case), sizes(256, case)
        assert narrow[0] > limits[0] and (wide[0] > limits[0]) == (tile == 128), case
        assert sizes(0, case) == (narrow if tile == 128 else wide), case
    narrowed = held_back = 0
    for case in cases:
        chosen, wide = sizes(0, case), sizes(256, case)
        if wide[0] <= limits[0] - 65536 and wide[1] <= limits[1]:
            assert chosen[0] <= limits[0] and chosen[1] <= limits[1], case
            narrow = sizes(128, case)
            narrowed += chosen == narrow != wide
            held_back += narrow[1] > limits[1] and chosen == wide != narrow   # by their partial results
    assert narrowed >= 5 and held_back >= 1
