"""The tile loop of the kernels with more than 32 query rows per work item: scores of one 32-key
half are formed while the previous half is exponentiated and the one before is multiplied with
its values, and a row's reference moves only when a half's probabilities outgrow it.  Key counts
around the 32-key halves and 64-key tiles, and keys that grow so that references have to move in
the first tile, between tiles and in a partial last half."""
import numpy as np
import pytest
import torch

from oracle import efim_oracle as O
from paper_2505_21889_amd import workloads as W

import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_21889_amd import binding
    return binding


# (cached, new): visible keys of the last row 33, 64, 65, 96, 97, 128, 129, 193, 321, 40
EDGES = ([0, 0, 1, 32, 33, 64, 65, 129, 257, 0], [33, 64, 64, 64, 64, 64, 64, 64, 64, 40])


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grow", [(), (32,), (64, 128), (40, 96, 190)])
def test_half_tile_edges_and_growing_scores(E, row_tile, d, grow):
    b = W.make_batch("c1", seed=4000 + d + len(grow), lengths=tuple(np.array(x, dtype=np.int32) for x in EDGES),
                     heads=(4, 2), head_dim=d)
    q_roped, kc, vc = U.oracle_inputs(b)
    # every key from position `at` on four times as large (an exact power of two in bf16): scores
    # of standard deviation 4, 16, 64 outgrow any reference taken before
    k = kc.reshape(b.cache_shape())
    for at in grow:
        for r in range(b.batch):
            for pos in range(at, int(b.cached_len[r] + b.new_len[r])):
                row = k[b.block_table[r, pos // b.page_size], :, pos % b.page_size]
                row[...] = np.where(row & 0x7F80, row + np.uint16(2 << 7), row)
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    try:
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
    # (a sharpened softmax gives outputs as large as single value rows: bound per element)
    U.assert_close(got, ref, "grow %s" % (grow,), large_outputs=True)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("heads", [(4, 4), (16, 2)])
@pytest.mark.parametrize("d", [64, 128])
def test_normaliser_is_the_sum_of_the_weights_used(E, row_tile, heads, d):
    """With every value element equal to 3 a row's output is 3 * (sum of the weights) / (row sum):
    exactly 3 when the row sum is taken over the very weights the value product uses (fp32 sums of
    at most 321 of them differ by under 1e-5, bf16 has 3 +- 7.8e-3 as neighbours).  Rows with few
    visible keys, whose weights carry 16 bits, included."""
    b = W.make_batch("c1", seed=4100 + d, lengths=tuple(np.array(x, dtype=np.int32) for x in EDGES),
                     heads=heads, head_dim=d)
    q_roped, kc, vc = U.oracle_inputs(b)
    vc[...] = 0x4040  # 3.0
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    try:
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
    assert np.all(got == 0x4040)


@pytest.mark.parametrize("page", [8, 16, 32, 64, 256])
@pytest.mark.parametrize("d", [64, 128])
def test_last_tile_of_few_rows_on_every_page_size(E, page, d):
    """At most 32 query rows: the last key tile of the range is gathered in groups of loads whose
    rows past the range repeat its last row.  Last tiles of 1 .. 64 keys; cache slots behind a
    request's end hold NaN patterns."""
    new = [1, 2, 3, 7, 8, 5, 3, 8, 6, 1, 8, 4, 8]
    ends = [1, 2, 8, 9, 15, 16, 17, 31, 33, 47, 48, 63, 64]
    cached = [64 * (i % 3) + e - n if 64 * (i % 3) + e >= n else 0 for i, (e, n) in enumerate(zip(ends, new))]
    b = W.make_batch("c1", seed=4200 + d + page, heads=(4, 2), head_dim=d, page_size=page,
                     lengths=(np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)))
    q_roped, kc, vc = U.oracle_inputs(b)
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    U.assert_close(U.gpu_extend_attention(E, b, q_roped, kc, vc), ref, "page %d" % page, large_outputs=True)


@pytest.mark.parametrize("parts", [2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("d", [64, 128])
def test_merge_kernel_for_every_group_of_parts(E, parts, d):
    """The merge reads two, four or eight parts at once; 20 tokens of two heads are 40 rows per
    item, past the in-kernel merge, in row blocks of 16 or 32."""
    b = W.make_batch("c1", seed=4300 + d, heads=(4, 2), head_dim=d,
                     lengths=(np.array([64 * parts - 20, 64 * parts - 33], dtype=np.int32), np.array([20, 13], dtype=np.int32)))
    q_roped, kc, vc = U.oracle_inputs(b)
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 64)
    try:
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    U.assert_close(got, ref, "%d parts" % parts)


@pytest.mark.parametrize("page", [8, 16, 32, 64, 256])
@pytest.mark.parametrize("new,row_tile", [([1, 2, 3, 7, 8, 5, 16, 4], 0), ([33, 64, 40, 7, 100, 65, 1, 20], 128),
                                          ([33, 64, 40, 7, 300, 65, 1, 20], 256)])
def test_code_rows_of_64_bytes_on_every_page_size(E, page, new, row_tile):
    """8-bit cache with head dim 64: one load takes sixteen rows, a page or several of them -- or two
    pages of eight, the one layout whose rows are looked up lane by lane.  Full and partial tiles,
    with few rows per item (first batch) and many."""
    from test_gpu_fp8 import gpu_attention8, oracle_cache8, oracle_step8
    cached = [0, 63, 200, 57, 128, 450, 15, 300]
    b = W.make_batch("c1", seed=4400 + page, heads=(4, 2), head_dim=64, page_size=page,
                     lengths=(np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)))
    k_scale, v_scale = 0.0123, 0.031
    q_roped, kc, vc, ref = oracle_step8(b, *oracle_cache8(b, k_scale, v_scale), k_scale, v_scale)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    try:
        got = gpu_attention8(E, b, q_roped, kc, vc, k_scale, v_scale)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
    U.assert_close(got, ref, "page %d" % page)
