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


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("d", [64, 128])
def test_weights_are_rounded_relative_to_the_first_tiles_maximum(E, row_tile, d):
    """A weight is bf16(2^(s - m)), m the row's maximum over the first 64 keys of its range (none of
    these scores outgrows it by 2^8), and an output is the rounded quotient of the fp32 sums.  In 64
    bits the same definition gives the same bf16 number unless a sum or an exponential falls
    within its fp32 error of a rounding boundary: about 1e-6 of an element's 2^-8 spacing for the
    sums, and one weight in 2000 rounded the other way shifts its row by 2^-8 / 64 at most -- under
    one element in a hundred.  Another reference rounds every weight elsewhere."""
    b = W.make_batch("c1", seed=4500 + d, heads=(4, 2), head_dim=d,
                     lengths=(np.array([20, 64, 150, 257], dtype=np.int32), np.array([50, 64, 64, 64], dtype=np.int32)))
    q_roped, kc, vc = U.oracle_inputs(b)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 0)
    try:
        got = O.bf16_to_f64(U.gpu_extend_attention(E, b, q_roped, kc, vc))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    scale = np.log2(np.e) / np.sqrt(d)
    differ, at = 0, 0
    for r in range(b.batch):
        c, n = int(b.cached_len[r]), int(b.new_len[r])
        for h in range(4):
            q = O.bf16_to_f64(q_roped[at:at + n, h])
            k, v = (O.gather_kv(x.reshape(b.cache_shape()), b.block_table[r], c + n, b.page_size, h // 2) for x in (kc, vc))
            k, v = (x if x.dtype == np.float64 else O.bf16_to_f64(x) for x in (k, v))
            s = q @ k.T * scale
            s[np.arange(c + n)[None, :] > c + np.arange(n)[:, None]] = -np.inf
            m = s[:, :64].max(axis=1, keepdims=True)
            assert (s.max(axis=1, keepdims=True) < m + 8).all()
            w = O.bf16_to_f64(O.f64_to_bf16(np.exp2(s - m)))
            out = O.bf16_to_f64(O.f64_to_bf16(w @ v / w.sum(axis=1, keepdims=True)))
            differ += int((out != got[at:at + n, h]).sum())
        at += n
    assert differ <= got.size // 100, "%d of %d elements" % (differ, got.size)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("d", [64, 128])
def test_weights_stay_in_range_of_the_largest_values(E, row_tile, d):
    """Values of 2^115: with weights of at most 2^8 their products stay far inside fp32.  Keys whose
    scores lie 2^13 and 2^15 above those of all keys before them move the reference instead of
    getting such a weight."""
    b = W.make_batch("c1", seed=4600 + d, heads=(4, 2), head_dim=d,
                     lengths=(np.array([100, 230], dtype=np.int32), np.array([64, 64], dtype=np.int32)))
    q_roped, kc, vc = U.oracle_inputs(b)
    q_roped[...] = 0
    q_roped[..., 0] = 0x3F80  # 1.0
    k = kc.reshape(b.cache_shape())
    for r in range(b.batch):
        total = int(b.cached_len[r] + b.new_len[r])
        for pos in range(total):
            grown = {70: 13.0, 77: 13.0, 200: 28.0, 225: 28.0}.get(pos, 0.0)
            k[b.block_table[r, pos // b.page_size], :, pos % b.page_size, 0] = O.f64_to_bf16(
                np.array([grown * np.sqrt(d) / np.log2(np.e)]))[0]
    v = O.bf16_to_f64(vc)
    vc[...] = np.where(np.isnan(v), vc, O.f64_to_bf16(np.where(np.isnan(v), 0.0, v) * 2.0 ** 115))
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 0)
    try:
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    U.assert_close(got, ref, large_outputs=True, value_scale=2.0 ** 115)


@pytest.mark.parametrize("parts", [9, 12, 17, 33])
@pytest.mark.parametrize("d", [64, 128])
def test_merges_of_more_than_eight_parts_agree_to_the_bit(E, parts, d):
    """Past eight parts the running sums are rescaled between groups: the merge kernel and the merge
    inside the attention kernel round that product, then add with one rounding."""
    b = W.make_batch("c1", seed=4700 + d, heads=(32, 8), head_dim=d,
                     lengths=(np.array([64 * parts - 8, 64 * parts - 40, 64 * parts - 20], dtype=np.int32),
                              np.array([8, 5, 7], dtype=np.int32)))
    q_roped, kc, vc = U.oracle_inputs(b)
    got = []
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 64)
    try:
        for inside in (0, 1):
            E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, inside)
            got.append(U.gpu_extend_attention(E, b, q_roped, kc, vc))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("row_tile", [0, 128, 256])
@pytest.mark.parametrize("split", [0, 64, 128])
@pytest.mark.parametrize("d", [64, 128])
def test_minus_infinity_scores_in_front_of_low_ones(E, row_tile, split, d):
    """Cached keys with minus infinity in an element that every query has at one: their scores are
    minus infinity, weight zero, over 32 .. 150 keys from the first on.  The scores behind lie 400
    log2 units below zero: relative to any reference but their own they vanish.  Row tile 0 with few
    rows takes the key-parallel kernel."""
    new = [5, 8, 3, 16, 12] if row_tile == 0 else [64, 64, 70, 64, 64]
    first_finite = [32, 40, 64, 100, 150]
    b = W.make_batch("c1", seed=4800 + d, heads=(4, 2), head_dim=d,
                     lengths=(np.array([170, 200, 330, 180, 250], dtype=np.int32), np.array(new, dtype=np.int32)))
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
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    U.assert_close(got, ref)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("grow", [(), (40, 96, 190)])
@pytest.mark.parametrize("page", [8, 16, 256])
def test_packed_kernel_gives_the_plain_kernels_bits(E, row_tile, grow, page):
    """Head dim 64 over a bf16 cache has a second form of the kernel, taken when there are many work
    items for the compute units; told that there is one unit, the planner takes it for any batch.
    Same arithmetic, so the same bits; lengths at the edges of halves and tiles, and keys that move
    references.  The plain form is compared with the oracle above."""
    b = W.make_batch("c1", seed=4900 + len(grow), heads=(8, 2), head_dim=64, page_size=page,
                     lengths=tuple(np.array(x, dtype=np.int32) for x in EDGES))
    q_roped, kc, vc = U.oracle_inputs(b)
    k = kc.reshape(b.cache_shape())
    for at in grow:
        for r in range(b.batch):
            for pos in range(at, int(b.cached_len[r] + b.new_len[r])):
                row = k[b.block_table[r, pos // b.page_size], :, pos % b.page_size]
                row[...] = np.where(row & 0x7F80, row + np.uint16(2 << 7), row)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    got = []
    try:
        for split in (0, 64):
            E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
            for slots in (0, 2):
                E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, slots)
                got.append(U.gpu_extend_attention(E, b, q_roped, kc, vc))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[2], got[3])
    U.assert_close(got[1], O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc),
                   large_outputs=True)


@pytest.mark.parametrize("page", [8, 16, 256])
@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("split", [-1, 64])
def test_short_step_over_code_rows_of_64_bytes(E, page, row_tile, split):
    """One launch over an 8-bit cache with head dim 64: full tiles and last tiles of 1 .. 64 keys, on pages
    of 8 (two pages to a load) and larger ones; codes byte for byte."""
    from test_gpu_fp8 import oracle_cache8, oracle_step8, run_decode8
    new = [1, 2, 7, 8, 5, 3, 8, 4]
    ends = [1, 9, 64, 65, 128, 200, 321, 700]
    cached = [max(0, e - n) for e, n in zip(ends, new)]
    b = W.make_batch("c1", seed=4950 + page, heads=(8, 2), head_dim=64, page_size=page,
                     lengths=(np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)))
    k_scale, v_scale = 0.0123, 0.031
    kc, vc = oracle_cache8(b, k_scale, v_scale)
    _, kc_ref, vc_ref, ref = oracle_step8(b, kc, vc, k_scale, v_scale)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        got, kc_got, vc_got, _ = run_decode8(E, b, kc, vc, k_scale, v_scale)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
    U.assert_close(got, ref, large_outputs=True)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("split", [0, 64, 128])
def test_growing_scores_through_split_ranges_and_codes(E, row_tile, d, cache, split):
    """Keys four times as large from positions 40, 96 and 190 on, so that references move inside a part and
    parts with very different references are merged; bf16 rows and codes (all below saturation)."""
    from test_gpu_fp8 import gpu_attention8, oracle_cache8
    from oracle import fp8_oracle as F
    b = W.make_batch("c1", seed=4970 + d, lengths=tuple(np.array(x, dtype=np.int32) for x in EDGES), heads=(4, 2), head_dim=d)
    scale = 1.0
    if cache == "bf16":
        q_roped, kc, vc = U.oracle_inputs(b)
        low, step = np.uint16(0x7F80), np.uint16(2 << 7)  # exponent field, factor of four
    else:
        kc, vc = oracle_cache8(b, scale, scale)
        q_roped, _ = F.rope_append_fp8(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new,
                                       kc, vc, b.rope_base, scale, scale)
        low, step = np.uint8(0x78), np.uint8(2 << 3)
    k = kc.reshape(b.cache_shape())
    for at in (40, 96, 190):
        for r in range(b.batch):
            for pos in range(at, int(b.cached_len[r] + b.new_len[r])):
                row = k[b.block_table[r, pos // b.page_size], :, pos % b.page_size]
                row[...] = np.where(row & low, row + step, row)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        if cache == "bf16":
            ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
            got = U.gpu_extend_attention(E, b, q_roped, kc, vc)
        else:
            ref = F.extend_attention_fp8(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc, scale, scale)
            got = gpu_attention8(E, b, q_roped, kc, vc, scale, scale)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    U.assert_close(got, ref, large_outputs=True)


@pytest.mark.parametrize("page", [8, 16, 256])
@pytest.mark.parametrize("split", [0, 64, 128])
def test_short_step_with_two_and_with_three_stages(E, page, split):
    """Head dim 64, bf16 cache, 128-row tiles: the short step takes a third stage when there are many work
    items for the compute units (here: told that there is one unit).  Ranges of 1 .. 11 tiles; the same bits
    and the same cache, against the oracle too."""
    from test_gpu_decode import oracle_step, run_decode
    new = [1, 2, 7, 8, 5, 3, 8, 4]
    ends = [1, 9, 64, 65, 129, 200, 321, 700]
    cached = [max(0, e - n) for e, n in zip(ends, new)]
    b = W.make_batch("c1", seed=4990 + page, heads=(8, 2), head_dim=64, page_size=page,
                     lengths=(np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)))
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 128)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    got = []
    try:
        for slots in (0, 2):
            E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, slots)
            out, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
            assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
            got.append(out)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
    assert np.array_equal(got[0], got[1])
    U.assert_close(got[0], ref, large_outputs=True)
