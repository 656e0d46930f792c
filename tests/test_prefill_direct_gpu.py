"""GPU parity of prefill's per-request single pass (a tile holds rows of one
request and reads its group's prefix itself), of the plan without tiles (a
workgroup per row and head; nested groups and fp32 too) and of the plan the
library picks by itself, against the oracle."""
import pytest

from gpu_util import assert_close, oracle_prefill_for, run_prefill, to_np, workspace_untouched
from test_prefill_gpu import device_dict, prefill_case, say
from workloads import make_batch, make_prefill_queries

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("setting", ["2", ""])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64)])
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "long_rows", "many_runs", "single"])
def test_prefill_direct_parity(kind, dtype, D, setting, monkeypatch):
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", setting)
    say("prefill direct", kind, dtype, D, repr(setting))
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=8)
    q, off = make_prefill_queries(plan, qr, seed=8)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    if setting == "2":
        assert workspace_untouched(keep[0]), "the split path ran"
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"direct {kind} {dtype} D={D}")


@pytest.mark.parametrize("dtype,D", [("float16", 64), ("bfloat16", 128), ("float32", 64),
                                     ("float32", 128)])
@pytest.mark.parametrize("kind", ["mixed", "wide_group", "nested", "long_rows", "many_runs", "single"])
def test_prefill_rows_parity(kind, dtype, D, monkeypatch):
    monkeypatch.setenv("PARROT_PREFILL_SINGLE_PASS", "3")
    say("prefill rows", kind, dtype, D)
    plan, qr = prefill_case(kind, dtype, D)
    batch = make_batch(plan, seed=9)
    q, off = make_prefill_queries(plan, qr, seed=9)
    keep = []
    out, lse = run_prefill(plan, device_dict(batch, q, off), off, keep=keep)
    assert workspace_untouched(keep[0]), "a tiled plan ran"
    ref = oracle_prefill_for(batch, plan, q, off)
    assert_close(*to_np(out, lse), *ref, dtype, f"rows {kind} {dtype} D={D}")
