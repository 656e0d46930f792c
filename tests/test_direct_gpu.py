"""GPU parity of the one-launch decode path of small calls (a workgroup per
request and head attends to the whole context and writes the output) where its
split can go wrong: contexts that end at a block, at the last wave's block (128
tokens with eight waves, 64 with four) or one token to either side, empty own
contexts, up to four prefix levels, both workgroup sizes, every entry point and
dtype, against the oracle.  The path is forced where the choice by size is not
the point; the poisoned workspace must come back untouched, which shows that it
ran."""
import math

import numpy as np
import pytest
import torch

from gpu_util import assert_close, decode_path, oracle_for, problem_for, run_gpu, to_np
from paper_2405_19888_amd import Decoder, parrot_shared_prefix_decode_noalloc
from workloads import build_plan, make_batch

pytestmark = pytest.mark.gpu

OWN = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 0, 33, 200]


def small_plan(dtype, D, heads, parents, seed=0):
    prefix = [65, 16, 63, 1][:len(parents)]
    gid = [(i % len(parents)) if s == 0 or i % 3 else -1 for i, s in enumerate(OWN)]
    return build_plan(heads=heads, head_dim=D, block_size=16, dtype=dtype, group_of_request=gid,
                      prefix_lens=prefix, suffix_lens=OWN, sm_scale=1.0 / math.sqrt(D), shuffle=True,
                      rng=np.random.default_rng(seed), prefix_parents=parents)


def check(plan, dev, batch, what, **kw):
    dec = Decoder(problem_for(plan))
    out, lse = run_gpu(plan, dev, decoder=dec, **kw)
    assert bool(torch.all(dec.workspace == 0xFF).item()), f"{what}: the two-kernel path ran"
    assert_close(*to_np(out, lse), *oracle_for(batch, plan), plan.dtype, what)
    return out.clone(), lse.clone()


@pytest.mark.parametrize("heads", [3, 24])                     # 42 and 336 workgroups
@pytest.mark.parametrize("parents", [[-1, -1, -1, -1], [-1, 0, 1, 2]])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", ["float16", "bfloat16", "float32"])
def test_direct_parity(dtype, D, parents, heads):
    what = f"direct {dtype} D={D} parents={parents} heads={heads}"
    print("[case]", what, flush=True)
    plan = small_plan(dtype, D, heads, parents)
    batch = make_batch(plan, seed=4)
    dev = batch.to("cuda")
    if heads == 24:          # eight waves above one workgroup per CU
        with decode_path("one8"):
            check(plan, dev, batch, what + " eight waves")
    with decode_path("one"):
        out, lse = check(plan, dev, batch, what)
    if not plan.nested:
        o2, l2 = torch.empty_like(out), torch.empty_like(lse)
        prob = problem_for(plan)
        with decode_path("one"):
            check(plan, dev, batch, what + " per request", shared=False)
            parrot_shared_prefix_decode_noalloc(
                prob, dev["q"], dev["k_pool"], dev["v_pool"], dev["k_pool"], dev["v_pool"],
                dev["prefix_tables"], dev["prefix_lens"], dev["suffix_tables"], dev["suffix_lens"],
                dev["group_ids"], o2, l2)
        torch.cuda.synchronize()
        assert torch.equal(out, o2) and torch.equal(lse, l2)


@pytest.mark.parametrize("heads", [3, 24])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("float32", 64)])
def test_direct_append(dtype, D, heads):
    """The new tokens reach the cache and the result is that of writing them
    first, bit for bit."""
    print("[case] direct append", dtype, D, heads, flush=True)
    plan = small_plan(dtype, D, heads, [-1, -1, -1, -1], seed=1)
    batch = make_batch(plan, seed=6)
    dev = batch.to("cuda")
    want_k, want_v = dev["k_pool"].clone(), dev["v_pool"].clone()
    R = plan.num_requests
    k_new, v_new = (torch.zeros(R, heads, D, dtype=want_k.dtype, device="cuda") for _ in range(2))
    for r in range(R):
        s = int(plan.suffix_lens[r])
        if s:
            b, t = int(plan.suffix_tables[r][(s - 1) // 16]), (s - 1) % 16
            k_new[r], v_new[r] = want_k[b, :, t], want_v[b, :, t]
            dev["k_pool"][b, :, t] = float("nan")
            dev["v_pool"][b, :, t] = float("nan")
    dev["k_new"], dev["v_new"] = k_new, v_new
    dec = Decoder(problem_for(plan))
    dec.workspace.fill_(0xFF)
    with decode_path("one"):
        out, lse = dec(dev, append=True)
    torch.cuda.synchronize()
    assert bool(torch.all(dec.workspace == 0xFF).item()), "the two-kernel path ran"
    out, lse = out.clone(), lse.clone()
    # bit patterns: unused slots hold NaN
    as_int = torch.int32 if dtype == "float32" else torch.int16
    assert torch.equal(dev["k_pool"].view(as_int), want_k.view(as_int))
    assert torch.equal(dev["v_pool"].view(as_int), want_v.view(as_int))
    with decode_path("one"):
        o2, l2 = dec(dev)
    torch.cuda.synchronize()
    assert torch.equal(out, o2) and torch.equal(lse, l2)
    assert_close(*to_np(out, lse), *oracle_for(batch, plan), dtype, "direct append")


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("dtype,D", [("float16", 128), ("bfloat16", 64), ("float32", 64)])
def test_direct_nonfinite(dtype, D, bad):
    """NaN or infinite inputs reach the output and the log-sum-exp: only an empty
    context gives 0 and -inf."""
    print("[case] direct nonfinite", dtype, D, bad, flush=True)
    plan = small_plan(dtype, D, 3, [-1, -1, -1, -1], seed=2)
    batch = make_batch(plan, seed=7)
    dev = batch.to("cuda")
    r = len(OWN) - 1
    dev["q"][r] = bad                       # every key of this request: NaN or mixed infinite logits
    dec = Decoder(problem_for(plan))
    dec.workspace.fill_(0xFF)
    with decode_path("one"):
        out, lse = dec(dev)
    torch.cuda.synchronize()
    assert bool(torch.all(dec.workspace == 0xFF).item()), "the two-kernel path ran"
    assert bool(torch.isnan(out[r]).all()) and bool(torch.isnan(lse[r]).all())
    rest = [i for i in range(plan.num_requests) if i != r]
    want, want_lse = oracle_for(batch, plan)
    assert_close(*to_np(out[rest], lse[rest]), want[rest], want_lse[rest], dtype, "direct nonfinite")
