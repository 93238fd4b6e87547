"""Launches with more work items than start at once, none of which share keys: the later ones are drawn from a
counter.  Every launch has to take each item once and to leave the counter at zero for the next, also beside the
arrival counters of cut ranges, over 8-bit caches and while another launch runs."""
import functools

import numpy as np
import pytest
import torch

from oracle import efim_oracle as O
from paper_2505_21889_amd import workloads as W

import gpu_util as U
from test_gpu_decode import oracle_step, run_decode
from test_gpu_fp8 import gpu_attention8, oracle_cache8, oracle_step8, run_decode8

pytestmark = pytest.mark.gpu

UNITS = 16   # compute units the planner is told to balance for, so that few items are more than start at once


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_21889_amd import binding
    return binding


@pytest.fixture(params=[(128, 0), (256, 0), (128, -1), (128, 2048), (256, 2048)], ids=lambda p: "tile%d split%d" % p)
def knobs(E, request):
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 2 * UNITS)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, request.param[0])
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, request.param[1])
    yield request.param
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
    E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, -1)
    E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)


def batch(pairs, most_new, d):
    """About `pairs` (request, kv head) pairs with 8 kv heads of 62 to 64 key tiles, and the pairs of a request of one tile
    and of one without new tokens."""
    rng = np.random.default_rng(pairs + most_new + d)
    n = rng.integers(1, most_new + 1, size=pairs // 8 + 2).astype(np.int32)
    c = rng.integers(3960, 4097 - most_new, size=len(n)).astype(np.int32)
    c[1] = 30
    n[2] = 0
    return W.make_batch("c1", seed=pairs + most_new + d, lengths=(c, n), heads=(8, 8), head_dim=d)


@functools.lru_cache(maxsize=None)
def inputs(pairs, most_new, d):
    b = batch(pairs, most_new, d)
    q, kc, vc = U.oracle_inputs(b)
    b.k_hist = b.v_hist = None
    return b, q, kc, vc, O.extend_attention(b.cached_len, b.new_len, b.block_table, b.page_size, q, kc, vc)


def draws(E, b, split, fp8=False):
    """Asserts that a launch over this batch draws items; with cut ranges that it also merges parts."""
    table = torch.from_numpy(b.block_table).cuda()
    info = E.efim_plan_info(U.make_desc(E, b, table), fp8)
    assert info["draws"] > info["queued_items"] > 0
    assert (info["merges"] > 0) == (split > 0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("pairs,most_new", [(4 * UNITS + 1, 40), (5 * UNITS + 9, 20), (6 * UNITS + 8, 3)])
def test_every_item_once_and_again(E, knobs, pairs, most_new, d):
    b, q, kc, vc, ref = inputs(pairs, most_new, d)
    draws(E, b, knobs[1])
    for merge in (-1, 0, 1) if knobs[1] > 0 else (-1,):
        E.efim_set_tuning(E.EFIM_TUNE_FUSED_MERGE, merge)
        first = U.gpu_extend_attention(E, b, q, kc, vc)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 0)   # items by workgroup id
        dealt = U.gpu_extend_attention(E, b, q, kc, vc)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)
        assert np.array_equal(first, dealt)
        for _ in range(2):
            assert np.array_equal(U.gpu_extend_attention(E, b, q, kc, vc), first)
        U.assert_close(first, ref, large_outputs=True)


@pytest.mark.parametrize("tile,split", [(128, 0), (256, 0), (128, 3840)])
@pytest.mark.parametrize("d", [64, 128])
def test_items_over_codes(E, d, tile, split):
    """8-bit caches draw items of 56 tiles and more in the mean, with more than 16 rows: both calls."""
    rng = np.random.default_rng(d + tile)
    n = rng.integers(9, 17, size=10).astype(np.int32)
    c = (rng.integers(3960, 4060, size=10) if split == 0 else np.full(10, 2 * 3840 - 20)).astype(np.int32)
    b = W.make_batch("c1", seed=d, lengths=(c, n), heads=(16, 8), head_dim=d)
    kc, vc = oracle_cache8(b, 0.0123, 0.031)
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 2 * UNITS)
    E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, tile)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, split)
    try:
        draws(E, b, split, fp8=True)
        q, kc_ref, vc_ref, ref = oracle_step8(b, kc, vc, 0.0123, 0.031)
        want = gpu_attention8(E, b, q, kc_ref, vc_ref, 0.0123, 0.031)
        U.assert_close(want, ref, large_outputs=True)
        step, kc_got, vc_got, _ = run_decode8(E, b, kc, vc, 0.0123, 0.031)
        assert np.array_equal(step, want) and np.array_equal(kc_got, kc_ref) and np.array_equal(vc_got, vc_ref)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 0)   # items by workgroup id
        assert np.array_equal(gpu_attention8(E, b, q, kc_ref, vc_ref, 0.0123, 0.031), want)
        assert np.array_equal(run_decode8(E, b, kc, vc, 0.0123, 0.031)[0], want)
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)
        E.efim_set_tuning(E.EFIM_TUNE_ROW_TILE, 0)
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)


def test_plan_object_launched_again_and_captured(E, knobs):
    """Plan objects draw nothing (their items follow the workgroup ids): launches in a row and replays of a graph, with
    other work between, against the batch call, which draws."""
    rng = np.random.default_rng(9)
    c = rng.integers(4000, 4096, size=5 * UNITS // 8 + 3).astype(np.int32)
    b = W.make_batch("c1", seed=9, lengths=(c, np.ones_like(c)), heads=(8, 8), head_dim=64)
    draws(E, b, knobs[1])
    kc, vc = U.oracle_cache(b)
    _, kc_ref, vc_ref, ref = oracle_step(b, kc, vc)
    want = run_decode(E, b, kc, vc)[0]
    U.assert_close(want, ref, large_outputs=True)
    table = torch.from_numpy(b.block_table).cuda()
    desc = U.make_desc(E, b, table)
    plan = E.Plan(desc, decode=True)
    nbytes = E.efim_plan_workspace_bytes(plan)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    q, kn, vn = U.dev_bits(b.q_new), U.dev_bits(b.k_new), U.dev_bits(b.v_new)
    kcd, vcd, out = U.dev_bits(kc), U.dev_bits(vc), torch.zeros_like(q)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        E.efim_plan_upload(plan, ws, nbytes, stream)

        def launch():
            E.efim_decode_step_planned(plan, table, q, kn, vn, kcd, vcd, out, b.rope_base, 0, 0.0, ws, stream)
        for _ in range(3):
            out.zero_()
            launch()
            stream.synchronize()
            assert np.array_equal(U.host_bits(out), want)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            launch()
        for _ in range(3):
            out.zero_()
            graph.replay()
            stream.synchronize()
            assert np.array_equal(U.host_bits(out), want)
            launch()
            stream.synchronize()
            assert np.array_equal(U.host_bits(out), want)
    assert np.array_equal(U.host_bits(kcd), kc_ref) and np.array_equal(U.host_bits(vcd), vc_ref)


def test_two_streams_at_once(E):
    """More items than the device starts at once; all requests read the same few pages.  Batch calls, which draw items,
    may run at the same time with a workspace each.  Launches of a plan whose ranges are whole only read its workspace:
    they may run at the same time with the same one, on two streams or as branches of one graph."""
    requests, heads, d, keys, page = 40, 32, 128, 2000, 16
    per = keys // page
    gen = torch.Generator(device="cuda").manual_seed(13)
    q = torch.randn(requests, heads, d, dtype=torch.bfloat16, device="cuda", generator=gen)
    k, v = (torch.randn(per, heads, page, d, dtype=torch.bfloat16, device="cuda", generator=gen) for _ in range(2))
    table = torch.arange(per, dtype=torch.int32).repeat(requests, 1).cuda()
    desc = E.BatchDesc([keys - 1] * requests, [1] * requests, table, heads, heads, d, page, per)
    E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, 0)
    E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 0)   # items by workgroup id
    try:
        want = torch.zeros_like(q)
        nbytes = E.efim_extend_workspace_bytes(desc)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        E.efim_extend_attention(desc, q, k, v, want, 0.0, ws, nbytes)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)
        items, info = E.efim_extend_plan_items(desc), E.efim_plan_info(desc)
        plan = E.Plan(desc)
        main, streams = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(2)]
        outs = [[torch.zeros_like(q) for _ in range(10)] for _ in range(2)]
        spaces = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        for i in range(10):
            for s, o, w in zip(streams, outs, spaces):
                E.efim_extend_attention(desc, q, k, v, o[i], 0.0, w, nbytes, s)
        torch.cuda.synchronize()
    finally:
        E.efim_set_tuning(E.EFIM_TUNE_SPLIT_KV, -1)
        E.efim_set_tuning(E.EFIM_TUNE_XCD_GROUPING, 1)
    assert len(items) == requests * heads and (items["partial_slot"] < 0).all()
    assert info["draws"] > info["queued_items"] > 0 and info["merges"] == 0
    for x, o in enumerate(outs):
        for i in range(10):
            assert torch.equal(o[i], want), "batch call: stream %d launch %d" % (x, i)
            o[i].zero_()
    some = [torch.nn.functional.softmax(k[:, h].reshape(keys, d).float() @ q[r, h].float() / d ** 0.5, 0) @
            v[:, h].reshape(keys, d).float() - want[r, h].float() for r, h in ((0, 0), (17, 5), (39, 31))]
    assert max(float(x.abs().max()) for x in some) <= U.MAX_ABS_TOL
    nbytes = E.efim_plan_workspace_bytes(plan)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    E.efim_plan_upload(plan, ws, nbytes)
    torch.cuda.synchronize()

    def both():
        for s in streams:
            s.wait_stream(main)
        for i in range(10):
            for s, o in zip(streams, outs):
                E.efim_extend_attention_planned(plan, table, q, k, v, o[i], 0.0, ws, s)
        for s in streams:
            main.wait_stream(s)

    def check(what):
        torch.cuda.synchronize()
        for x, o in enumerate(outs):
            for i in range(10):
                assert torch.equal(o[i], want), "%s: stream %d launch %d" % (what, x, i)
                o[i].zero_()
        torch.cuda.synchronize()

    both()
    check("two streams")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=main):
        both()
    for replay in range(3):
        graph.replay()
        check("replay %d" % replay)
