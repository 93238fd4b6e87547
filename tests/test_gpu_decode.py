"""The fused step (decode: one new token per request; short steps: up to 16 new tokens and 32
query rows per kv head) against the oracle's rope_append followed by its extend_attention, and
against the library's own two-call path: caches bit-exact, q left untouched, outputs within the
attention tolerance and identical to the two-call path."""
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


def run_decode(E, b, kc, vc, interleaved=0, ws=None, sm_scale=0.0):
    table = torch.from_numpy(b.block_table).cuda()
    desc = U.make_desc(E, b, table)
    q = U.dev_bits(b.q_new)
    k_new, v_new = U.dev_bits(b.k_new), U.dev_bits(b.v_new)
    kcd, vcd = U.dev_bits(kc), U.dev_bits(vc)
    out = torch.full(q.shape, 0x7FC1, dtype=torch.int16, device="cuda")
    nbytes = E.efim_decode_workspace_bytes(desc)
    assert nbytes >= 256
    if ws is None:
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")   # contents must not matter
    assert ws.numel() >= nbytes
    E.efim_decode_step(desc, q, k_new, v_new, kcd, vcd, out, b.rope_base, interleaved, sm_scale, ws, ws.numel())
    torch.cuda.synchronize()
    assert np.array_equal(U.host_bits(q), b.q_new), "q must stay as given"
    return U.host_bits(out), U.host_bits(kcd), U.host_bits(vcd), ws


def oracle_step(b, kc, vc, interleaved=False):
    kc, vc = kc.copy(), vc.copy()
    q_roped, _ = O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new,
                               kc, vc, b.rope_base, interleaved)
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_roped, kc, vc)
    return q_roped, kc, vc, ref


def two_call_path(E, b, kc, vc, interleaved=0):
    table = torch.from_numpy(b.block_table).cuda()
    desc = U.make_desc(E, b, table)
    q = U.dev_bits(b.q_new)
    kcd, vcd = U.dev_bits(kc), U.dev_bits(vc)
    E.efim_rope_append(desc, q, U.dev_bits(b.k_new), U.dev_bits(b.v_new), kcd, vcd, b.rope_base, interleaved)
    out = torch.full(q.shape, 0x7FC1, dtype=torch.int16, device="cuda")
    nbytes = E.efim_extend_workspace_bytes(desc)
    ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    E.efim_extend_attention(desc, q, kcd, vcd, out, 0.0, ws, nbytes)
    torch.cuda.synchronize()
    return U.host_bits(out)


CASES = [
    # name,        cached lengths,                           heads,    D,  interleaved
    ("gqa_ragged", [0, 1, 15, 16, 17, 63, 64, 300, 1000, 2047], (8, 2), 128, 0),
    ("mha",        [5, 129, 640],                            (4, 4), 128, 0),
    ("gqa7_d128",  [777, 31, 4096],                          (28, 4), 128, 1),
    ("d64",        [0, 100, 1025, 48],                       (8, 4), 64, 0),
    ("d64_il",     [33, 2000],                               (4, 1), 64, 1),
]


@pytest.mark.parametrize("split", [-1, 64, 0])
@pytest.mark.parametrize("name,cached,heads,d,interleaved", CASES)
def test_decode_step_matches_oracle_and_two_call_path(E, name, cached, heads, d, interleaved, split):
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        c = np.array(cached, dtype=np.int32)
        b = W.make_batch("c1", seed=50 + len(cached), lengths=(c, np.ones_like(c)), heads=heads, head_dim=d)
        kc, vc = U.oracle_cache(b, fill=0x3C00 if name == "mha" else W.POISON_BITS)
        q_ref, kc_ref, vc_ref, ref = oracle_step(b, kc, vc, bool(interleaved))
        got, kc_got, vc_got, ws = run_decode(E, b, kc, vc, interleaved)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref), "cache append must be bit-exact"
        U.assert_close(got, ref, name)
        assert np.array_equal(got, two_call_path(E, b, kc, vc, interleaved)), "fused and two-call outputs differ"
        # a second step on the same workspace (the arrival counters were put back), same result
        got2, _, _, _ = run_decode(E, b, kc, vc, interleaved, ws=ws)
        assert np.array_equal(got, got2)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


SHORT_CASES = [
    # name,       cached lengths,                              new tokens,                   heads,   D,  interleaved
    # (cached lengths around multiples of 64: the new keys then lie in two key tiles, and with a
    #  forced split of 64 keys in two work items)
    ("mha_16",    [0, 1, 50, 63, 64, 100, 1000, 2047],          [16] * 8,                    (4, 4), 128, 0),
    ("mha_mixed", [5, 60, 127, 128, 640, 3000, 56, 0],          [1, 2, 3, 16, 7, 8, 5, 9],   (4, 4), 128, 0),
    ("gqa4",      [60, 63, 64, 56, 120, 0, 127, 4095],          [8, 1, 3, 4, 8, 2, 5, 7],    (8, 2), 128, 0),
    ("gqa7",      [777, 61, 4096, 0],                           [4, 1, 3, 2],                (28, 4), 128, 1),
    ("d64_g2",    [0, 100, 1025, 48, 62],                       [16, 9, 1, 12, 16],          (8, 4), 64, 0),
    ("d64_il",    [33, 2000, 190],                              [3, 11, 16],                 (4, 4), 64, 1),
]


@pytest.mark.parametrize("split", [-1, 64, 0])
@pytest.mark.parametrize("name,cached,new,heads,d,interleaved", SHORT_CASES)
def test_short_step_matches_oracle_and_two_call_path(E, name, cached, new, heads, d, interleaved, split):
    """Several new tokens per request in one launch: every new key is rotated, patched into the
    tiles that hold it and appended by exactly one workgroup of its kv head."""
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        c, n = np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)
        b = W.make_batch("c1", seed=150 + len(cached), lengths=(c, n), heads=heads, head_dim=d)
        kc, vc = U.oracle_cache(b)
        q_ref, kc_ref, vc_ref, ref = oracle_step(b, kc, vc, bool(interleaved))
        got, kc_got, vc_got, ws = run_decode(E, b, kc, vc, interleaved)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref), "cache append must be bit-exact"
        U.assert_close(got, ref, name)
        assert np.array_equal(got, two_call_path(E, b, kc, vc, interleaved)), "fused and two-call outputs differ"
        got2, _, _, _ = run_decode(E, b, kc, vc, interleaved, ws=ws)
        assert np.array_equal(got, got2)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


@pytest.mark.parametrize("name,cached,new,heads,d,interleaved", [SHORT_CASES[1], SHORT_CASES[4]])
def test_short_step_in_the_eight_wave_configuration(E, name, cached, new, heads, d, interleaved):
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 256)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 128)
    try:
        c, n = np.array(cached, dtype=np.int32), np.array(new, dtype=np.int32)
        b = W.make_batch("c1", seed=170 + len(cached), lengths=(c, n), heads=heads, head_dim=d)
        kc, vc = U.oracle_cache(b)
        _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc, bool(interleaved))
        got, kc_got, vc_got, _ = run_decode(E, b, kc, vc, interleaved)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, name)
        assert np.array_equal(got, two_call_path(E, b, kc, vc, interleaved))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


@pytest.mark.parametrize("row_tile", [128, 256])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [(4, 4), (8, 4), (6, 1)])
def test_rows_of_an_item_at_the_edges_of_the_write_out(E, heads, d, row_tile):
    """1 .. 32 query rows per item (the write-out takes 8, 16 or 32 rows at a time), written directly and as
    parts, the parts combined in either way."""
    g = heads[0] // heads[1]
    n = np.array([t for t in (1, 2, 4, 5, 8, 9, 15, 16) if t * g <= 32], dtype=np.int32)
    c = np.array([70 + 33 * i for i in range(len(n))], dtype=np.int32)
    b = W.make_batch("c1", seed=190 + d + g, lengths=(c, n), heads=heads, head_dim=d)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    try:
        for split in (0, 64):
            outs = []
            for fused in (0, 1):
                E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
                E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, fused)
                got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
                assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
                U.assert_close(got, ref, "split %d merge %d" % (split, fused))
                outs.append(got)
            assert np.array_equal(outs[0], outs[1])
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)


@pytest.mark.parametrize("page_size", [8, 16, 256])
@pytest.mark.parametrize("heads,d", [((8, 2), 128), ((4, 4), 128), ((8, 2), 64)])
def test_ranges_gathered_at_once(E, heads, d, page_size):
    """Few items of few rows: key ranges of one tile up to all that the buffers hold, one key more (a split range),
    ends just in front of, on and behind tile edges, new tokens in one tile, over an edge and over a
    split; in one call and as two calls, over bf16 rows and codes."""
    from test_gpu_fp8 import oracle_cache8, oracle_step8, run_decode8
    most = 64 * (4 if d == 128 else 8)
    ends = [1, 5, 64, 65, 130, most - 60, most - 1, most, most + 1, 2 * most + 3]
    n = [1, 5, 3, 4, 8, 2, 7, 8, 4, 8]
    c = np.array([e - k for e, k in zip(ends, n)], dtype=np.int32)
    n = np.array(n, dtype=np.int32)
    b = W.make_batch("c1", seed=210 + d + page_size, lengths=(c, n), heads=heads, head_dim=d, page_size=page_size)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
    assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
    U.assert_close(got, ref, large_outputs=True)
    assert np.array_equal(got, two_call_path(E, b, kc, vc))
    k_scale, v_scale = 0.0123, 0.031
    kc, vc = oracle_cache8(b, k_scale, v_scale)
    _, kc_ref, vc_ref, ref = oracle_step8(b, kc, vc, k_scale, v_scale)
    got, kc_got, vc_got, _ = run_decode8(E, b, kc, vc, k_scale, v_scale)
    assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
    U.assert_close(got, ref, large_outputs=True)


@pytest.mark.parametrize("row_tile,split", [(0, -1), (128, 64), (256, 64)])
@pytest.mark.parametrize("page_size", [8, 16, 256])
@pytest.mark.parametrize("heads,d", [((3, 3), 128), ((16, 1), 128), ((4, 2), 64)])
def test_sixteen_rows_per_item(E, heads, d, page_size, row_tile, split):
    """Launches whose largest item has exactly 16 query rows: first and last rows and keys of both 16-key
    blocks of a half tile, in every form of the kernel, over bf16 rows and codes."""
    from test_gpu_fp8 import oracle_cache8, oracle_step8, run_decode8
    g = heads[0] // heads[1]
    n = np.array([max(1, 16 // g), 1, max(1, 8 // g), 1, 1], dtype=np.int32)
    c = np.array([113, 15, 16, 48, 700], dtype=np.int32)
    b = W.make_batch("c1", seed=230 + d + g + page_size, lengths=(c, n), heads=heads, head_dim=d, page_size=page_size)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, row_tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        kc, vc = U.oracle_cache(b)
        _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
        got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, large_outputs=True)
        assert np.array_equal(got, two_call_path(E, b, kc, vc))
        kc, vc = oracle_cache8(b, 0.0123, 0.031)
        _, kc_ref, vc_ref, ref = oracle_step8(b, kc, vc, 0.0123, 0.031)
        got, kc_got, vc_got, _ = run_decode8(E, b, kc, vc, 0.0123, 0.031)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, large_outputs=True)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


@pytest.mark.parametrize("page_size", [8, 256])
def test_short_step_other_page_sizes(E, page_size):
    c = np.array([0, 7, 8, 60, 64, 250, 256, 1000, 2049], dtype=np.int32)
    n = np.array([8, 2, 8, 7, 1, 8, 3, 6, 8], dtype=np.int32)
    b = W.make_batch("c1", seed=140 + page_size, lengths=(c, n), heads=(8, 2), head_dim=128, page_size=page_size)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    for split in (-1, 64):
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
        try:
            got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
        finally:
            E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, "page %d split %d" % (page_size, split))


@pytest.mark.parametrize("name,cached,heads,d,interleaved", [CASES[0], CASES[3]])
def test_decode_step_in_the_eight_wave_configuration(E, name, cached, heads, d, interleaved):
    """The 256-row launch configuration (chosen by the planner for large batches; forced here)."""
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 256)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 128)
    try:
        c = np.array(cached, dtype=np.int32)
        b = W.make_batch("c1", seed=70 + len(cached), lengths=(c, np.ones_like(c)), heads=heads, head_dim=d)
        kc, vc = U.oracle_cache(b)
        _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc, bool(interleaved))
        got, kc_got, vc_got, _ = run_decode(E, b, kc, vc, interleaved)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, name)
        assert np.array_equal(got, two_call_path(E, b, kc, vc, interleaved))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


@pytest.mark.parametrize("page_size", [8, 64, 256])
def test_decode_step_other_page_sizes(E, page_size):
    c = np.array([0, 7, 8, 63, 64, 255, 256, 1000, 2049], dtype=np.int32)
    b = W.make_batch("c1", seed=40 + page_size, lengths=(c, np.ones_like(c)), heads=(8, 2), head_dim=128,
                     page_size=page_size)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    for split in (-1, 64):
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
        try:
            got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
        finally:
            E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        U.assert_close(got, ref, "page %d split %d" % (page_size, split))


def test_decode_merge_across_compute_dies(E):
    """With the planner's XCD grouping off the parts of a split key range land on different
    dies: the merging workgroup must still see every partial result."""
    E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 0)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 64)
    try:
        c = np.array([3000, 4500, 900, 2222, 5000, 64], dtype=np.int32)
        b = W.make_batch("c1", seed=77, lengths=(c, np.ones_like(c)), heads=(16, 4), head_dim=128)
        kc, vc = U.oracle_cache(b)
        _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
        ws = None
        for rep in range(3):
            got, kc_got, vc_got, ws = run_decode(E, b, kc, vc, ws=ws)
            assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
            U.assert_close(got, ref, "rep %d" % rep)
            assert np.array_equal(got, two_call_path(E, b, kc, vc))
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)


def test_in_kernel_merge_soak_on_three_streams(E):
    """A bounded soak of the hand-over between the workgroups of a split key range: 360 decode
    steps queued on three streams, XCD grouping off (the parts of a range land on different dies),
    every key range cut into 64-key parts, merge inside the kernel; every output compared bit for
    bit with what the separate merge kernel gives.  Stops at the first mismatch."""
    c = np.array([3000, 4500, 900, 2222, 5000, 64, 1777, 333], dtype=np.int32)
    b = W.make_batch("c1", seed=78, lengths=(c, np.ones_like(c)), heads=(16, 4), head_dim=128)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 0)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 64)
    try:
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, 0)
        want, _, _, _ = run_decode(E, b, kc, vc)
        U.assert_close(want, ref, "second-launch merge")
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, 1)
        table = torch.from_numpy(b.block_table).cuda()
        desc = U.make_desc(E, b, table)
        q, k_new, v_new = U.dev_bits(b.q_new), U.dev_bits(b.k_new), U.dev_bits(b.v_new)
        nbytes = E.efim_decode_workspace_bytes(desc)
        streams = [torch.cuda.Stream() for _ in range(3)]
        lanes = []
        for s_ in streams:   # every stream has its own caches, output and workspace
            lanes.append((s_, U.dev_bits(kc), U.dev_bits(vc), [torch.empty_like(q) for _ in range(8)],
                          torch.empty(nbytes, dtype=torch.uint8, device="cuda")))
        torch.cuda.synchronize()
        for rnd in range(15):
            for s_, kcd, vcd, outs, ws in lanes:
                for o in outs:
                    E.efim_decode_step(desc, q, k_new, v_new, kcd, vcd, o, b.rope_base, 0, 0.0, ws, nbytes, s_)
            torch.cuda.synchronize()
            for li, (s_, kcd, vcd, outs, ws) in enumerate(lanes):
                for oi, o in enumerate(outs):
                    assert np.array_equal(U.host_bits(o), want), "round %d stream %d step %d" % (rnd, li, oi)
        for s_, kcd, vcd, outs, ws in lanes:
            assert np.array_equal(U.host_bits(kcd), kc_ref) and np.array_equal(U.host_bits(vcd), vc_ref)
            E.efim_stream_release(s_)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)


def test_decode_step_with_the_merge_in_a_second_launch(E):
    """The decode step also works when the parts of a split key range are combined by the
    separate merge kernel (the path taken when a launch has more split tiles than arrival
    counters): same bits as the in-kernel merge."""
    c = np.array([2500, 700, 4100], dtype=np.int32)
    b = W.make_batch("c1", seed=61, lengths=(c, np.ones_like(c)), heads=(8, 2), head_dim=128)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 512)
    try:
        in_kernel, _, _, _ = run_decode(E, b, kc, vc)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, 0)
        second_launch, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)
    assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
    U.assert_close(second_launch, ref, "second launch")
    assert np.array_equal(in_kernel, second_launch)


@pytest.mark.parametrize("merges", [511, 512, 1024, 4095, 4096, 8191, 8192])
def test_as_many_split_ranges_as_there_are_counters(E, merges):
    """Arrival counters lie further apart the fewer a launch needs; 8192 split ranges are one more than a launch has
    counters.  Batch call and plan object, each twice, against the oracle, and bit for bit against the second launch."""
    c = np.full(merges, 100, dtype=np.int32)
    b = W.make_batch("c1", seed=merges, lengths=(c, np.ones_like(c)), heads=(1, 1), head_dim=64)
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 64)
    try:
        table = torch.from_numpy(b.block_table).cuda()
        desc = U.make_desc(E, b, table)
        assert E.efim_plan_info(desc)["merges"] == merges
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, 0)
        want = run_decode(E, b, kc, vc)[0]
        U.assert_close(want, ref)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, 1)
        for _ in range(2):
            got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
            assert np.array_equal(got, want) and np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        plan = E.Plan(desc, decode=True)
        nbytes = E.efim_plan_workspace_bytes(plan)
        ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
        E.efim_plan_upload(plan, ws, nbytes)
        q, kn, vn, kcd, vcd = (U.dev_bits(x) for x in (b.q_new, b.k_new, b.v_new, kc, vc))
        for _ in range(2):
            out = torch.zeros_like(q)
            E.efim_decode_step_planned(plan, table, q, kn, vn, kcd, vcd, out, b.rope_base, 0, 0.0, ws)
            assert np.array_equal(U.host_bits(out), want)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)


def test_decode_sequence_grows_the_cache_token_by_token(E):
    """Eight consecutive decode steps of three requests: the caches after the last step and
    every step's output equal the oracle's, which appends token by token too."""
    heads, d = (8, 2), 128
    c0 = np.array([14, 250, 1023], dtype=np.int32)
    steps = 8
    first = W.make_batch("c1", seed=91, lengths=(c0, np.ones_like(c0)), heads=heads, head_dim=d)
    # a block table with room for all steps, shared by all of them
    roomy = W.make_batch("c1", seed=91, lengths=(c0, np.full_like(c0, steps)), heads=heads, head_dim=d,
                         with_history=True)
    kc, vc = U.oracle_cache(roomy)
    kc_ref, vc_ref = kc.copy(), vc.copy()
    kc_dev, vc_dev = kc.copy(), vc.copy()
    # one workspace for the whole sequence; the plans of the steps differ
    ws = torch.full((8 << 20,), 0x5A, dtype=torch.uint8, device="cuda")
    for s in range(steps):
        b = W.make_batch("c1", seed=200 + s, lengths=(c0 + s, np.ones_like(c0)), heads=heads, head_dim=d,
                         with_history=False)
        b.block_table, b.num_pages = roomy.block_table, roomy.num_pages
        q_ref, kc_ref, vc_ref, ref = oracle_step(b, kc_ref, vc_ref)
        got, kc_dev, vc_dev, ws = run_decode(E, b, kc_dev, vc_dev, ws=ws)
        assert np.array_equal(kc_dev, kc_ref) and np.array_equal(vc_dev, vc_ref), "step %d" % s
        U.assert_close(got, ref, "step %d" % s)


def test_decode_shapes_of_the_benchmark(E):
    """Decode at the batch shapes of c2 / c3 (cached lengths as drawn for those workloads)."""
    for base in ("c2", "c3"):
        spec = W.make_batch(base, with_history=False, with_tensors=False)
        b = W.make_batch(base, lengths=(spec.cached_len, np.ones_like(spec.new_len)))
        kc, vc = U.oracle_cache(b)
        _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
        got, kc_got, vc_got, _ = run_decode(E, b, kc, vc)
        assert np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        max_abs, rel = U.assert_close(got, ref, base)
        print("%s decode: max_abs %.3e rel_l2 %.3e" % (base, max_abs, rel))


def test_decode_step_rejects_other_batches(E):
    c = np.array([10, 20], dtype=np.int32)
    lib = E.raw_library()
    import ctypes
    fake = 0x10000
    # a request without a new token, with more than 16 of them, with more than 32 query rows per kv head
    for new, heads in (([1, 0], (4, 4)), ([1, 17], (4, 4)), ([1, 5], (8, 1)), ([9, 1], (8, 2))):
        b = W.make_batch("c1", lengths=(c, np.array(new, dtype=np.int32)), heads=heads, head_dim=64)
        table = torch.from_numpy(b.block_table).cuda()
        desc = U.make_desc(E, b, table)
        assert E.efim_decode_workspace_bytes(desc) == 0
        rc = lib.efim_decode_step(ctypes.byref(desc.c), fake, fake, fake, fake, fake, fake + 0x1000, 1e4, 0, 0.0, fake, 1 << 20, None)
        assert rc == E.EFIM_ERR_UNSUPPORTED, (new, heads)
    b1 = W.make_batch("c1", lengths=(c, np.ones_like(c)), heads=(4, 4), head_dim=64)
    desc1 = U.make_desc(E, b1, torch.from_numpy(b1.block_table).cuda())
    need = E.efim_decode_workspace_bytes(desc1)
    assert need > 0
    rc = lib.efim_decode_step(ctypes.byref(desc1.c), fake, fake, fake, fake, fake, fake + 0x1000, 1e4, 0, 0.0, fake, need - 1, None)
    assert rc == E.EFIM_ERR_WORKSPACE
    rc = lib.efim_decode_step(ctypes.byref(desc1.c), fake, fake, fake, fake, fake, fake + 0x1000, 1e4, 2, 0.0, fake, need, None)
    assert rc == E.EFIM_ERR_INVALID_ARG


@pytest.mark.parametrize("d,rotary_dim,interleaved,heads", [(128, 128, 0, (8, 2)), (128, 64, 0, (8, 2)), (128, 32, 1, (28, 4)),
                                                           (64, 64, 1, (4, 4)), (64, 16, 0, (8, 4)), (128, 96, 1, (4, 1))])
def test_decode_step_with_a_frequency_table(E, d, rotary_dim, interleaved, heads):
    """efim_decode_step_table: a caller-given frequency table (the Llama 3.1 long-context scaling)
    and rotation of the leading rotary_dim elements only -- caches bit for bit, output within the
    bar and identical to efim_rope_append_table followed by efim_extend_attention."""
    c = np.array([0, 31, 32, 63, 700, 2047, 4100], dtype=np.int32)
    b = W.make_batch("c1", seed=95 + rotary_dim, lengths=(c, np.ones_like(c)), heads=heads, head_dim=d)
    table = O.scaled_inv_freq(rotary_dim, 5.0e5, 8.0, 1.0, 4.0, 8192)
    kc, vc = U.oracle_cache(b)
    kc_ref, vc_ref = kc.copy(), vc.copy()
    q_ref, _ = O.rope_append_table(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new,
                                   kc_ref, vc_ref, table, rotary_dim, bool(interleaved))
    ref = O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q_ref, kc_ref, vc_ref)
    tab = torch.from_numpy(b.block_table).cuda()
    desc = U.make_desc(E, b, tab)
    q, kcd, vcd = U.dev_bits(b.q_new), U.dev_bits(kc), U.dev_bits(vc)
    out = torch.full(q.shape, 0x7FC1, dtype=torch.int16, device="cuda")
    nbytes = E.efim_decode_workspace_bytes(desc)
    ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    E.efim_decode_step_table(desc, q, U.dev_bits(b.k_new), U.dev_bits(b.v_new), kcd, vcd, out, table, rotary_dim,
                             interleaved, 0.0, ws, nbytes)
    torch.cuda.synchronize()
    assert np.array_equal(U.host_bits(q), b.q_new), "q must stay as given"
    assert np.array_equal(U.host_bits(kcd), kc_ref) and np.array_equal(U.host_bits(vcd), vc_ref)
    U.assert_close(U.host_bits(out), ref, "rotary_dim %d" % rotary_dim)
    # the two-call path on the same inputs
    q2, kc2, vc2 = U.dev_bits(b.q_new), U.dev_bits(kc), U.dev_bits(vc)
    E.efim_rope_append_table(desc, q2, U.dev_bits(b.k_new), U.dev_bits(b.v_new), kc2, vc2, table, rotary_dim, interleaved)
    out2 = torch.full(q.shape, 0x7FC1, dtype=torch.int16, device="cuda")
    nb2 = E.efim_extend_workspace_bytes(desc)
    ws2 = torch.empty(max(nb2, 256), dtype=torch.uint8, device="cuda")
    E.efim_extend_attention(desc, q2, kc2, vc2, out2, 0.0, ws2, nb2)
    torch.cuda.synchronize()
    assert np.array_equal(U.host_bits(out), U.host_bits(out2)), "fused and two-call outputs differ"


def test_decode_step_table_rejects_bad_tables(E):
    c = np.array([10, 20], dtype=np.int32)
    b = W.make_batch("c1", lengths=(c, np.ones_like(c)), heads=(4, 4), head_dim=64)
    desc = U.make_desc(E, b, torch.from_numpy(b.block_table).cuda())
    good = O.rope_inv_freq(64, 1e4)
    for table, rotary_dim in ((good, 8), (good, 24), (np.ones(64), 128), (np.full(32, np.nan), 64), (np.full(32, np.inf), 64)):
        with pytest.raises(E.EfimError):
            E.efim_decode_step_table(desc, 1, 1, 1, 1, 1, 2, table, rotary_dim, 0, 0.0, 1, 256)
