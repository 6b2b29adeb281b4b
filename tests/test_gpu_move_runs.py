"""What is dealt out over the whole chip from per-unit counts: an eviction's moves and the segments that change hands."""
import numpy as np
import pytest

from tests.test_gpu_evict_sizes import _check

pytestmark = pytest.mark.gpu


# the long units first, last and in between; in a thousand, one in 97 and the last
@pytest.mark.parametrize("units,long", [(1, [0]), (9, [0]), (9, [4]), (9, [8]), (1024, list(range(5, 1024, 97)) + [1023])])
def test_moves_of_units_with_very_different_lists(units, long):
    """Units with some thousand moves beside units with a few or none."""
    lengths = [4000 if i in long else 300 + i % 5 for i in range(units)]
    budgets = [n // 2 if i in long else (n if i % 3 else n - 7) for i, n in enumerate(lengths)]
    evicted = np.subtract(lengths, budgets)
    assert (evicted == 2000).sum() == len(long) and (units == 1 or ((evicted == 0).any() and (evicted == 7).any()))
    _check(units, 4032, lengths, budgets, None, sorted(set(long) | set(range(0, units, 1 if units < 10 else 89))), False)


@pytest.mark.parametrize("units,cap,edge", [(4, 24608, [12288, 12289, 24576, 24577]), (300, 8160, [3072, 3073, 6144, 6145])])
@pytest.mark.parametrize("n_sink", [None, 20])
def test_widths_between_the_powers_of_two(units, cap, edge, n_sink):
    """Twelve and twenty-four entries per thread, of 1024 and of 256."""
    lengths = [edge[i % 4] for i in range(units)]
    budgets = [max(1, n - 1 - (i * 371) % (n - 1)) for i, n in enumerate(lengths)]
    _check(units, cap, lengths, budgets, n_sink, range(0, units, 1 + units // 12), False)


def _deal(own, rows, spare, need):
    """Segments as the definition deals them out: surplus of units in order to the stack, then what units lack from its top."""
    for u in range(len(own)):
        spare += [rows[u][j] for j in range(need[u], own[u])]
        rows[u] = rows[u][:min(own[u], need[u])]
    if sum(max(0, need[u] - own[u]) for u in range(len(own))) > len(spare):
        return False
    for u in range(len(own)):
        while len(rows[u]) < need[u]:
            rows[u].append(spare.pop())
    return True


@pytest.mark.parametrize("short", [False, True])
@pytest.mark.parametrize("units", [3, 1023, 1024, 1025, 2500])
def test_segments_are_dealt_as_defined(units, short):
    from paper_2601_16986_amd import ckv
    rng = np.random.default_rng(units)
    cap = 3072
    old = rng.integers(1, cap - 64, (1, units, 1)).astype(np.int32)
    g = ckv.CrystalKV(1, units, 1, 1, 128, cap, old, t0=1, headroom=1, budget_min=1, budget_max=cap - 2)
    seg = lambda b: (b.reshape(-1) + 1 + 255) // 256
    before = g.segment_table()
    rows = [list(before["rows"][u, :before["owned"][u]]) for u in range(units)]
    spare = list(before["spare"])
    # the same budgets dealt to other units, or (short) more than the pools hold
    new = np.full_like(old, cap - 2) if short else rng.permutation(old.reshape(-1)).reshape(old.shape)
    g.set_budgets(new)
    g.rebalance()
    enough = _deal(list(before["owned"]), rows, spare, seg(new))
    assert enough != short and bool(g.status() & 4) == short
    after = g.segment_table()
    assert np.array_equal(after["owned"], [len(r) for r in rows])
    for u in range(units):
        assert list(after["rows"][u, :len(rows[u])]) == rows[u] and not after["rows"][u, len(rows[u]):].any()
    assert list(after["spare"]) == spare
    g.close()
