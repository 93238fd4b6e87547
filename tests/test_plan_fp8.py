"""The plans of batch calls over 8-bit caches (no GPU: planning is host code)."""
import numpy as np
import pytest

from paper_2505_21889_amd import binding as E


@pytest.fixture(autouse=True)
def slots():
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 512)
    yield
    E.efim_set_tuning(E.EFIM_TUNE_NUM_SLOTS, 0)


def desc(cached, new, heads, d=128):
    pages = -(-(np.array(cached) + np.array(new)) // 16)
    return E.BatchDesc(cached, new, np.zeros((len(cached), int(pages.max())), np.int32), heads[0], heads[1], d, 16, 1 << 24)


STEPS = {
    "bound by HBM, more than 128 rows": ([5000] * 32, [30] * 32, (28, 4)),
    "few rows": ([3000] * 8, [4] * 8, (8, 2)),
    "compute-heavy, short ranges": ([1000] * 16, [256] * 16, (32, 8)),
    "compute-heavy, long ranges": ([16384] * 4, [512] * 4, (32, 8)),
}


@pytest.mark.parametrize("step", STEPS)
def test_one_plan_where_the_format_does_not_change_the_tile(step):
    """The size query's plan serves the call, unless a call over 8-bit caches takes another tile."""
    d = desc(*STEPS[step])
    need = E.efim_extend_workspace_bytes(d)
    before = E.efim_plan_info(d)
    after = E.efim_plan_info(d, fp8=True)
    assert (after["plans_built"] == before["plans_built"]) == (step != "compute-heavy, long ranges")
    assert after["row_tile"] == 128 and before["row_tile"] == (256 if step == "compute-heavy, long ranges" else 128)
    for _ in range(3):
        assert E.efim_plan_info(d, fp8=True) == after
        assert E.efim_extend_workspace_bytes(d) == need


def test_the_plan_fits_what_the_query_said():
    """Over drawn compute-heavy steps whose tiles differ: 128 rows unless they need more workspace than the query says,
    which a buffer of exactly that size has to do."""
    rng = np.random.default_rng(17)
    own = other = 0
    for _ in range(150):
        batch = int(rng.integers(1, 9))
        d = desc(rng.integers(2000, 16000, batch).tolist(), rng.integers(40, 400, batch).tolist(),
                 [(32, 8), (28, 4)][int(rng.integers(0, 2))])
        need, plain, info = E.efim_extend_workspace_bytes(d), E.efim_plan_info(d), E.efim_plan_info(d, fp8=True)
        assert info["workspace_bytes"] <= need and plain["workspace_bytes"] == need
        if plain["row_tile"] == 256:
            own += info["row_tile"] == 128
            other += info["row_tile"] == 256
    assert own >= 20 and other >= 3
