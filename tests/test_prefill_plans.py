"""Which plan prefill takes for calls of plain sizes (CPU: the choice reads host
scalars only; 256 compute units are assumed without a GPU)."""
import ctypes

import pytest

from paper_2405_19888_amd import binding as B


def choice(requests, heads, prefix, rows, own=None, nested=False, dtype=1):
    own = own or rows
    groups = 1 if prefix else 0
    prob = B.make_problem(
        num_requests=requests, num_heads=heads, head_dim=128, block_size=16, num_groups=groups,
        max_group_size=requests if groups else 0, max_prefix_len=prefix, max_suffix_len=own,
        prefix_table_stride=-(-prefix // 16), suffix_table_stride=-(-own // 16),
        num_prefix_blocks=4096, num_suffix_blocks=65536, dtype=dtype, sm_scale=0.1)
    t = B.make_prefill_rows(requests * rows, rows, requests * rows if groups else 0)
    return B.parrot_prefill_single_pass(prob, t, nested=nested)


@pytest.mark.parametrize("kw,single", [
    (dict(requests=1, heads=32, prefix=0, rows=300), True),       # 18 us split, 12 us in one pass
    (dict(requests=4, heads=32, prefix=0, rows=600), True),       # 59 / 30 us
    (dict(requests=1, heads=8, prefix=0, rows=4000), False),      # too few tiles: 65 / 102 us
    (dict(requests=16, heads=32, prefix=100, rows=40), True),     # 24 / 15 us
    (dict(requests=64, heads=32, prefix=600, rows=40), True),     # 104 / 59 us
    (dict(requests=64, heads=32, prefix=2000, rows=4, own=8), False),     # 51 / 113 us
    (dict(requests=64, heads=32, prefix=6000, rows=16, own=1000), False), # 215 us split
    (dict(requests=64, heads=32, prefix=6000, rows=559, own=1000), True),
])
def test_plan_by_sizes(parrot_lib, kw, single, monkeypatch):
    monkeypatch.delenv("PARROT_PREFILL_SINGLE_PASS", raising=False)
    assert choice(**kw) == single
    assert not choice(**kw, nested=True) and not choice(**kw, dtype=0)


SPLIT, STACKED, DIRECT, ROWS4, ROWS8 = 0, 1, 2, 3, 19       # ROWS8: eight waves per workgroup


@pytest.mark.parametrize("kw,plan", [
    # rows without tiles: the longest context and first reads of prefixes count
    (dict(requests=4, heads=4, head_dim=64, prefix=128, own=32, total=96, most=32, dtype=0), ROWS4),   # 18.5 us / 6.3
    (dict(requests=8, heads=8, prefix=200, own=40, total=8, most=1), ROWS8),                           # 14.1 / 5.9
    (dict(requests=4096, heads=8, prefix=200, own=40, total=8, most=1), ROWS8),                        # 55.8 / 6.1
    (dict(requests=2, heads=32, head_dim=64, groups=8, prefix=1405, own=5, total=10, most=5), SPLIT),  # 15.9 / 19.6
    (dict(requests=5, heads=4, prefix=17, own=1054, total=73, most=15), SPLIT),                        # 13.8 / 18.0
    # 57 of its groups unread
    (dict(requests=3, heads=8, head_dim=64, groups=60, prefix=2593, own=371, total=33, most=11), SPLIT),  # 39.3 / 46.5
    # one row each of 59 requests: 72 us split, 63 in tiles per request
    (dict(requests=59, heads=20, groups=12, prefix=152, own=2555, total=59, most=1, group_rows=10), DIRECT),
    (dict(requests=16, heads=32, prefix=100, own=64, total=640, most=64), DIRECT),                     # 24 / 26 / 15
    (dict(requests=64, heads=32, prefix=600, own=64, total=2560, most=64), STACKED),                   # 104 / 59 / 84
])
def test_plan_kinds(parrot_lib, kw, plan, monkeypatch):
    monkeypatch.delenv("PARROT_PREFILL_SINGLE_PASS", raising=False)
    k = dict(dict(groups=1, dtype=1, head_dim=128), **kw)
    prob = B.make_problem(
        num_requests=k["requests"], num_heads=k["heads"], head_dim=k["head_dim"], block_size=16, num_groups=k["groups"],
        max_group_size=1, max_prefix_len=k["prefix"], max_suffix_len=k["own"],
        prefix_table_stride=-(-k["prefix"] // 16), suffix_table_stride=-(-k["own"] // 16),
        num_prefix_blocks=65536, num_suffix_blocks=65536, dtype=k["dtype"], sm_scale=0.1)
    rows = B.make_prefill_rows(k["total"], k["most"], k.get("group_rows", k["total"]))
    assert parrot_lib.parrot_test_prefill_plan(ctypes.byref(prob), ctypes.byref(rows), 0) == plan
    if plan == SPLIT:
        assert not B.parrot_prefill_single_pass(prob, rows)
    else:
        assert B.parrot_prefill_single_pass(prob, rows)


def test_rows_plan_stays_within_one_launch(parrot_lib, monkeypatch):
    """Forced, the plan without tiles is left to calls whose workgroups one launch
    can hold (less than 2^32 threads)."""
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "3")
    for total, plan in ((1 << 17, ROWS4), (1 << 18, SPLIT)):
        prob = B.make_problem(
            num_requests=1 << 12, num_heads=32, head_dim=64, block_size=16, num_groups=0, max_group_size=0,
            max_prefix_len=0, max_suffix_len=100, prefix_table_stride=0, suffix_table_stride=7,
            num_prefix_blocks=1, num_suffix_blocks=65536, dtype=0, sm_scale=0.1)
        rows = B.make_prefill_rows(total, 100, 0)
        assert parrot_lib.parrot_test_prefill_plan(ctypes.byref(prob), ctypes.byref(rows), 0) == plan
