"""The key-parallel kernels, for launches whose work items have at most 32 query rows: products of
16 rows (no item has more) and of 32, over a ring of tile buffers and with the whole key range of an
item gathered at once.  Which of them a launch takes follows from the plan: forced splitting never
takes the whole-range kernel, and automatic splitting over few tiles does unless some range is of a
length that neither fits it nor is cut."""
import numpy as np
import pytest
import torch

from oracle import efim_oracle as O
from paper_2505_21889_amd import workloads as W

import gpu_util as U
from test_gpu_decode import oracle_step, run_decode, two_call_path
from test_gpu_fp8 import gpu_attention8, oracle_cache8, oracle_step8, run_decode8

pytestmark = pytest.mark.gpu

ONCE_TILES = {64: 8, 128: 4}   # key tiles that the whole-range kernel holds
K_SCALE, V_SCALE = 0.0123, 0.031


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_21889_amd import binding
    return binding


class _knobs:
    def __init__(self, E, row_tile=0, split=-1):
        self.E, self.values = E, (row_tile, split)

    def __enter__(self):
        self.E.efim_set_tuning(self.E.EFIM_TUNE_ROW_TILE, self.values[0])
        self.E.efim_set_tuning(self.E.EFIM_TUNE_SPLIT_KV, self.values[1])

    def __exit__(self, *exc):
        self.E.efim_set_tuning(self.E.EFIM_TUNE_ROW_TILE, 0)
        self.E.efim_set_tuning(self.E.EFIM_TUNE_SPLIT_KV, -1)


def planned(E, b):
    """(most rows of a work item, most key tiles of one) of the plan under the current knobs."""
    items = E.efim_extend_plan_items(U.make_desc(E, b, torch.from_numpy(b.block_table).cuda()))
    items = items[items["row_count"] > 0]
    return int(items["row_count"].max()), int((-(-(items["key_end"] - items["key_begin"]) // 64)).max())


def batch(seed, rows, ends, new, **more):
    """Requests of 8/2 heads with keys up to `ends`; `new` tokens each, capped so that an item has at most `rows`."""
    n = np.minimum(np.array(new, dtype=np.int32), rows // 4)
    c = np.array(ends, dtype=np.int32) - n
    return W.make_batch("c1", seed=seed, lengths=(c.astype(np.int32), n), heads=(8, 2), **more)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("page_size", [8, 16, 64, 256])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("d", [64, 128])
def test_ring_of_several_tiles(E, d, rows, page_size, row_tile):
    """Ranges of three tiles (which fill and wrap the buffers) and of up to eleven, last tiles of one row up to
    all, as one call and as two, over bf16 rows and codes."""
    b = batch(500 + d + page_size + rows, rows, [700, 193, 449, 192, 577, 640, 33], [8, 3, 8, 4, 1, 7, 5], head_dim=d,
              page_size=page_size)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    kc8, vc8 = oracle_cache8(b, K_SCALE, V_SCALE)
    q8, kc8_ref, vc8_ref, ref8 = oracle_step8(b, kc8, vc8, K_SCALE, V_SCALE)
    for split, tiles in ((192, 3), (640, 11)):
        with _knobs(E, row_tile, split):
            most, longest = planned(E, b)
            assert most == rows and longest >= tiles
            got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
            assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
            U.assert_close(got, ref, "split %d" % split)
            assert np.array_equal(got, two_call_path(E, b, kc, vc))
            got, kc_got, vc_got, _ = run_decode8(E, b, kc8, vc8, K_SCALE, V_SCALE)
            assert np.array_equal(kc_got, kc8_ref) and np.array_equal(vc_got, vc8_ref)
            U.assert_close(got, ref8, "codes, split %d" % split)
            assert np.array_equal(got, gpu_attention8(E, b, q8, kc8_ref, vc8_ref, K_SCALE, V_SCALE))


@pytest.mark.parametrize("row_tile,split", [(0, -1), (0, 0), (256, 0), (256, 512), (128, 128)])
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("d", [64, 128])
def test_growing_scores(E, d, rows, cache, row_tile, split):
    """Cached keys four times as large from four (codes: three) positions on.  References move from half to half of a
    ring; in the whole-range kernel they lie far apart between the eight waves, and with head dim 64
    also move inside a wave, which takes every fourth tile; split parts are merged.  (The codes stay below saturation.)"""
    ends = [21, 101, 250, 480, 330, 505, 700]
    b = batch(560 + d + rows, rows, ends, [1, 2, 8, 8, 3, 8, 5], head_dim=d)
    if cache == "bf16":
        kc, vc = U.oracle_cache(b)
        grow, low, step = (32, 96, 190, 290), np.uint16(0x7F80), np.uint16(2 << 7)  # exponent field, factor of four
    else:
        kc, vc = oracle_cache8(b, 1.0, 1.0)
        grow, low, step = (32, 96, 290), np.uint8(0x78), np.uint8(2 << 3)
    k = kc.reshape(b.cache_shape())
    for at in grow:
        for r in range(b.batch):
            for pos in range(at, int(b.cached_len[r])):
                row = k[b.block_table[r, pos // b.page_size], :, pos % b.page_size]
                row[...] = np.where(row & low, row + step, row)
    with _knobs(E, row_tile, split):
        most, longest = planned(E, b)
        assert most == rows and (longest <= ONCE_TILES[d] if split < 0 else longest >= split // 64)
        if cache == "bf16":
            _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
            got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
            plain = two_call_path(E, b, kc, vc)
        else:
            q8, kc_ref, vc_ref, ref = oracle_step8(b, kc, vc, 1.0, 1.0)
            got, kc_got, vc_got, _ = run_decode8(E, b, kc, vc, 1.0, 1.0)
            plain = gpu_attention8(E, b, q8, kc_ref, vc_ref, 1.0, 1.0)
    assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
    U.assert_close(got, ref, large_outputs=True)
    assert np.array_equal(got, plain)


@pytest.mark.parametrize("split", [-1, 0, 64])
@pytest.mark.parametrize("rows", [16, 32])
@pytest.mark.parametrize("d", [64, 128])
def test_minus_infinity_scores_in_front_of_low_ones(E, d, rows, split):
    """Cached keys with minus infinity in an element that every query has at one, from the first on over 32 .. 230 keys:
    waves and parts that see no other score, and such a half in front of scores 400 log2 units below
    zero, which vanish relative to any reference but their own."""
    first_finite = [32, 40, 64, 100, 150, 230, 0]
    b = batch(590 + d + rows, rows, [180, 210, 340, 190, 500, 250, 70], [1, 8, 3, 8, 5, 8, 2], head_dim=d)
    q_roped, kc, vc = U.oracle_inputs(b)
    q_roped[..., :2] = 0x3F80  # 1.0
    k = kc.reshape(b.cache_shape())
    low = O.f64_to_bf16(np.array([-400.0 * np.sqrt(d) / np.log2(np.e)]))[0]
    for r in range(b.batch):
        for pos in range(int(b.cached_len[r] + b.new_len[r])):
            row = k[b.block_table[r, pos // b.page_size], :, pos % b.page_size]
            row[:, 0] = 0xFF80 if pos < first_finite[r] else 0
            row[:, 1] = low
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    with _knobs(E, 0, split):
        most, longest = planned(E, b)
        assert most == rows and (longest <= ONCE_TILES[d] if split < 0 else longest >= split // 64)
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    U.assert_close(got, ref)
