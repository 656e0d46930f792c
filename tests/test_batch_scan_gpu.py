"""GPU parity of the two-kernel decode at request counts where its set-up scans
change: a wave's 64 requests, the four waves' steps, the member scan's 256 and
2048, one launch's 4096, each with one request fewer or more; own lengths with
runs of empty requests, groups spread over the batch, flat and nested.  A sample
of requests against the oracle, and every request against the per-request path
(other scans, no prefix role)."""
import math

import numpy as np
import pytest

from gpu_util import assert_close, decode_path, oracle_for, problem_for, run_gpu, to_np
from paper_2405_19888_amd import Decoder
from workloads import build_plan, make_batch

pytestmark = pytest.mark.gpu


COUNTS = [(R, n, "float16", 64) for R in (64, 65, 255, 257, 1025, 2049, 4096, 4097, 5000) for n in (False, True)]
COUNTS += [(65, False, "bfloat16", 128), (257, True, "bfloat16", 128), (65, True, "float32", 128),
           (257, False, "float32", 64)]


@pytest.mark.parametrize("R,nested,dtype,D", COUNTS)
def test_decode_request_counts(R, nested, dtype, D):
    print("[case] decode", R, "requests nested", nested, dtype, D, flush=True)
    rng = np.random.default_rng(R)
    heads = 8 if R < 300 else 2
    gid = rng.integers(0, 5, size=R)
    gid[gid == 4] = -1
    own = rng.integers(0, 70, size=R)
    own[rng.random(R) < 0.3] = 0
    own[(gid < 0) & (own == 0)] = 17
    plan = build_plan(heads=heads, head_dim=D, block_size=16, dtype=dtype,
                      group_of_request=gid.tolist(), prefix_lens=[2400, 1040, 33, 16],
                      prefix_parents=[-1, 0, 1, -1] if nested else None, suffix_lens=own.tolist(),
                      sm_scale=1.0 / math.sqrt(D), rng=rng)
    batch = make_batch(plan, seed=R)
    dev = batch.to("cuda")
    dec = Decoder(problem_for(plan))
    with decode_path("two"):
        out, lse = to_np(*run_gpu(plan, dev, decoder=dec))
    assert bool((dec.workspace != 0xFF).any().item()), "the one-launch path ran"
    assert np.all(np.isfinite(out)) and np.all(np.isfinite(lse))
    sample = sorted(set([0, 1, 63, R // 2, R - 2, R - 1]) | set(rng.integers(0, R, 24).tolist()))
    sample = [r for r in sample if 0 <= r < R]
    ref = oracle_for(batch, plan, requests=sample)
    pick = (lambda x: x[sample]) if ref[0].shape[0] == R else (lambda x: x)
    assert_close(out[sample], lse[sample], pick(ref[0]), pick(ref[1]), dtype, f"{R} requests")
    if not nested:
        with decode_path("two"):
            o2, l2 = to_np(*run_gpu(plan, dev, shared=False))
        assert_close(out, lse, o2, l2, dtype, f"{R} requests vs per request")
