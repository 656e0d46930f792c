"""Which plan prefill takes for calls of plain sizes (CPU: the choice reads host
scalars only; 256 compute units are assumed without a GPU)."""
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
