"""The append kernel where it can go wrong: the request table (64 requests per load, 384 per launch, requests
without new tokens), head layouts whose rows do not fill a wave's passes, the grid of large steps, and
results on the way from fp64 to bf16 whose fp32 form is a midpoint of two bf16 numbers."""
import numpy as np
import pytest
import torch

from oracle import efim_oracle as O
from paper_2505_21889_amd import workloads as W

import gpu_util as U
from oracle import fp8_oracle as F
from test_gpu_decode import run_decode
from test_gpu_fp8 import gpu_append8, oracle_cache8, oracle_step8, run_decode8

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_21889_amd import binding
    return binding


@pytest.mark.parametrize("batch", [1, 63, 64, 65, 128, 384, 385, 449])
def test_request_table(E, batch):
    rng = np.random.default_rng(batch)
    n = rng.integers(0, 3, size=batch).astype(np.int32)
    n[[0, batch // 2, -1]] = [2, 0, 1]
    c = rng.integers(0, 40, size=batch).astype(np.int32)
    b = W.make_batch("c1", seed=batch, lengths=(c, n), heads=(2, 1), head_dim=64)
    kc, vc = U.oracle_cache(b)
    got = U.gpu_rope_append(E, b, kc, vc)
    q_ref, _ = O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new, kc, vc,
                             b.rope_base)
    for x, y in zip(got, (q_ref, kc, vc)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("interleaved", [0, 1])
@pytest.mark.parametrize("heads,d", [((1, 1), 64), ((1, 1), 128), ((14, 1), 128), ((15, 1), 128), ((28, 4), 128),
                                     ((30, 2), 64), ((31, 1), 64), ((32, 32), 128), ((64, 8), 128)])
def test_head_layouts(E, heads, d, interleaved):
    """Rows of a token below, at and above what one, two, three and more waves take (16 rows of 128, 32 of 64)."""
    b = W.make_batch("c1", seed=heads[0] + d, lengths=(np.array([3, 0, 40], np.int32), np.array([5, 0, 9], np.int32)),
                     heads=heads, head_dim=d)
    kc, vc = U.oracle_cache(b)
    got = U.gpu_rope_append(E, b, kc, vc, interleaved)
    kc8, vc8 = oracle_cache8(b, 0.0123, 0.031)
    got8 = gpu_append8(E, b, kc8, vc8, 0.0123, 0.031, interleaved)
    q_ref, _ = O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new, kc, vc,
                             b.rope_base, interleaved=bool(interleaved))
    for x, y in zip(got, (q_ref, kc, vc)):
        assert np.array_equal(x, y)
    q8, kc8_ref, vc8_ref, _ = oracle_step8(b, kc8, vc8, 0.0123, 0.031, interleaved=bool(interleaved))
    for x, y in zip(got8, (q8, kc8_ref, vc8_ref)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("interleaved", [0, 1])
@pytest.mark.parametrize("heads,d", [((7, 1), 128), ((28, 4), 128), ((32, 8), 64), ((32, 32), 128)])
def test_keys_only(E, heads, d, interleaved):
    """Without queries a token has its key and value rows alone: one wave or several, and a wave that is not full."""
    b = W.make_batch("c1", seed=heads[0] + d, lengths=(np.array([3, 0, 40], np.int32), np.array([5, 0, 9], np.int32)),
                     heads=heads, head_dim=d)
    kc, vc = U.oracle_cache(b)
    kc8, vc8 = oracle_cache8(b, 0.0123, 0.031)
    _, *got = U.gpu_rope_append(E, b, kc, vc, interleaved, with_q=False)
    table = torch.from_numpy(b.block_table).cuda()
    got8 = [torch.from_numpy(x.copy()).cuda() for x in (kc8, vc8)]
    E.efim_rope_append_fp8(U.make_desc(E, b, table), None, U.dev_bits(b.k_new), U.dev_bits(b.v_new), *got8, b.rope_base,
                           interleaved, 0.0123, 0.031)
    O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, None, b.k_new, b.v_new, kc, vc, b.rope_base,
                  interleaved=bool(interleaved))
    _, kc8, vc8, _ = oracle_step8(b, kc8, vc8, 0.0123, 0.031, interleaved=bool(interleaved))
    for x, y in zip(got + [x.cpu().numpy() for x in got8], (kc, vc, kc8, vc8)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("heads,d", [((4, 1), 64), ((28, 4), 128)])
def test_large_step_equals_small_ones(E, heads, d):
    """A step of more than 512 MiB of head rows (workgroups of whole tokens; (4, 1): of four each) against the same
    tokens in steps that stay below, which the other tests compare with the oracle."""
    hq, hkv = heads
    total = (1 << 29) // ((hq + 2 * hkv) * d * 2) + 77
    n = [total // 3, total - total // 3]
    c = [5, 1000]
    page, dev = 16, "cuda"
    per = [-(-(x + y) // page) for x, y in zip(c, n)]
    pages = sum(per)
    gen = torch.Generator(device=dev).manual_seed(d)
    order = torch.randperm(pages, generator=torch.Generator().manual_seed(d)).to(torch.int32)
    table = torch.zeros(2, max(per), dtype=torch.int32)
    table[0, :per[0]], table[1, :per[1]] = order[:per[0]], order[per[0]:]
    table = table.to(dev)
    q0 = torch.randn(total, hq, d, dtype=torch.bfloat16, device=dev, generator=gen)
    k, v = (torch.randn(total, hkv, d, dtype=torch.bfloat16, device=dev, generator=gen) for _ in range(2))
    results = []
    for steps in (1, 3):
        q = q0.clone()
        kc, vc = (torch.zeros(pages, hkv, page, d, dtype=torch.bfloat16, device=dev) for _ in range(2))
        done = [0, 0]
        for s in range(steps):
            part = [x * (s + 1) // steps - y for x, y in zip(n, done)]
            for r in (0, 1) if steps > 1 else (None,):
                who = [0, 1] if r is None else [r]
                lo = 0 if r is None else (done[0] if r == 0 else n[0] + done[1])
                desc = E.BatchDesc([c[i] + done[i] for i in who], [part[i] for i in who],
                                   table if r is None else table[r:r + 1], hq, hkv, d, page, pages)
                hi = lo + sum(part[i] for i in who)
                E.efim_rope_append(desc, q[lo:hi], k[lo:hi], v[lo:hi], kc, vc, 1.0e6)
            done = [x + y for x, y in zip(done, part)]
        torch.cuda.synchronize()
        results.append((q, kc, vc))
    for x, y in zip(*results):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16))


def test_midpoints_round_once(E):
    """Values whose rotation lies next to a midpoint of two bf16 numbers, closer than fp32 can tell: searched for on
    the host, in fp64, among many pairs; each unit of eight pairs that has one takes the value-by-value path."""
    d, pos = 64, 11
    rng = np.random.default_rng(7)
    inv = 1.0e4 ** (-2.0 * np.arange(d // 2) / d)
    cos, sin = np.cos(pos * inv), np.sin(pos * inv)
    found = []
    for _ in range(40):
        x = O.f64_to_bf16(rng.standard_normal((20000, d)))
        f = O.bf16_to_f64(x)
        y1 = f[:, :d // 2] * cos - f[:, d // 2:] * sin
        low = y1.astype(np.float32).view(np.uint32) & 0xFFFF
        found.append(x[(low == 0x8000).any(axis=1)])
    rows = np.concatenate(found)
    assert len(rows) > 50
    rows = rows[:len(rows) // 4 * 4]
    b = W.make_batch("c1", seed=1, lengths=(np.full(len(rows) // 4, pos, np.int32), np.ones(len(rows) // 4, np.int32)),
                     heads=(4, 4), head_dim=d)
    b.rope_base = 1.0e4
    b.q_new[:] = rows.reshape(b.q_new.shape)
    b.k_new[:] = rows.reshape(b.k_new.shape)
    for interleaved in (0, 1):
        kc, vc = U.oracle_cache(b)
        if interleaved:
            swap = np.stack([np.arange(d // 2), np.arange(d // 2) + d // 2], axis=1).ravel()
            b.q_new[:] = b.q_new[..., swap]
            b.k_new[:] = b.k_new[..., swap]
        got = U.gpu_rope_append(E, b, kc, vc, interleaved)
        q_ref, _ = O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new, kc, vc,
                                 b.rope_base, interleaved=bool(interleaved))
        for x, y in zip(got, (q_ref, kc, vc)):
            assert np.array_equal(x, y)


SPECIAL = np.array([0x7F80, 0xFF80, 0x7FC0, 0xFFC0, 0x7F81, 0xFFFF, 0x0000, 0x8000, 0x0001, 0x8001, 0x007F, 0x0080, 0x8080,
                    0x00FF, 0x7F7F, 0xFF7F, 0x3F80, 0xBF80], np.uint16)   # inf, NaN, zero, subnormal, least normal, largest, one


@pytest.mark.parametrize("interleaved", [0, 1])
@pytest.mark.parametrize("heads,d", [((8, 2), 128), ((4, 4), 64)])
def test_special_values_are_rotated_as_in_fp64(E, heads, d, interleaved):
    """Infinities, NaN, zeros, subnormals and the largest numbers beside bit patterns drawn at random, as queries, keys
    and values: each number as the oracle has it, NaN (whose bits are not defined) where it has NaN."""
    rng = np.random.default_rng(d + interleaved)
    c, n = np.array([0, 5, 900], np.int32), np.array([8, 5, 8], np.int32)   # (position 0: cosine 1, sine 0)
    b = W.make_batch("c1", seed=d, lengths=(c, n), heads=heads, head_dim=d)
    for x in (b.q_new, b.k_new, b.v_new):
        x[:] = np.where(rng.random(x.shape) < 0.5, rng.choice(SPECIAL, x.shape), rng.integers(0, 1 << 16, x.shape))

    def same(got, want):
        nan = np.isnan(O.bf16_to_f64(want))
        assert np.array_equal(np.isnan(O.bf16_to_f64(got)), nan) and np.array_equal(got[~nan], want[~nan])

    with np.errstate(all="ignore"):
        kc, vc = U.oracle_cache(b)
        got = U.gpu_rope_append(E, b, kc, vc, interleaved)
        step = run_decode(E, b, kc, vc, interleaved)[1:3]
        q_ref, _ = O.rope_append(b.cached_len, b.new_len, b.block_table, b.page_size, b.q_new, b.k_new, b.v_new, kc, vc,
                                 b.rope_base, interleaved=bool(interleaved))
        assert np.isnan(O.bf16_to_f64(q_ref)).any() and np.isinf(O.bf16_to_f64(q_ref)).any()
        for x, y in zip(got + step, (q_ref, kc, vc, kc, vc)):
            same(x, y)
        for scale in (0.0123, 300.0, 2.0 ** -126, 3.0e38):
            kc8, vc8 = oracle_cache8(b, scale, scale)
            got = gpu_append8(E, b, kc8, vc8, scale, scale, interleaved)
            step = run_decode8(E, b, kc8, vc8, scale, scale, interleaved)[1:3]
            F.rope_append_fp8(b.cached_len, b.new_len, b.block_table, b.page_size, None, b.k_new, b.v_new, kc8, vc8,
                              b.rope_base, scale, scale, bool(interleaved))
            same(got[0], q_ref)
            for x, y in zip(got[1:] + step, (kc8, vc8, kc8, vc8)):   # (one code stands for every NaN)
                assert np.array_equal(x, y)
