"""GPU parity of the two-kernel decode at request counts where its set-up scans
change: a wave's 64 requests, the four waves' steps, the member scan's 256 and
2048, one launch's 4096, each with one request fewer or more; own lengths with
runs of empty requests, groups spread over the batch, flat and nested.  A sample
of requests against the oracle, and every request against the per-request path
(other scans, no prefix role)."""
import math

import numpy as np
import pytest

from gpu_util import assert_close, oracle_for, problem_for, run_gpu, to_np
from paper_2405_19888_amd import Decoder
from workloads import build_plan, make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nested", [False, True])
@pytest.mark.parametrize("R", [64, 65, 255, 257, 1025, 2049, 4096, 4097, 5000])
def test_decode_request_counts(R, nested):
    print("[case] decode", R, "requests nested", nested, flush=True)
    rng = np.random.default_rng(R)
    heads = 8 if R < 300 else 2                    # enough prefix reads to leave the one-launch path
    gid = rng.integers(0, 5, size=R)
    gid[gid == 4] = -1
    own = rng.integers(0, 70, size=R)
    own[rng.random(R) < 0.3] = 0
    own[(gid < 0) & (own == 0)] = 17
    plan = build_plan(heads=heads, head_dim=64, block_size=16, dtype="float16",
                      group_of_request=gid.tolist(), prefix_lens=[2400, 1040, 33, 16],
                      prefix_parents=[-1, 0, 1, -1] if nested else None, suffix_lens=own.tolist(),
                      sm_scale=1.0 / math.sqrt(64), rng=rng)
    batch = make_batch(plan, seed=R)
    dev = batch.to("cuda")
    dec = Decoder(problem_for(plan))
    out, lse = to_np(*run_gpu(plan, dev, decoder=dec))
    assert bool((dec.workspace != 0xFF).any().item()), "the one-launch path ran"
    assert np.all(np.isfinite(out)) and np.all(np.isfinite(lse))
    sample = sorted(set([0, 1, 63, R // 2, R - 2, R - 1]) | set(rng.integers(0, R, 24).tolist()))
    sample = [r for r in sample if 0 <= r < R]
    ref = oracle_for(batch, plan, requests=sample)
    pick = (lambda x: x[sample]) if ref[0].shape[0] == R else (lambda x: x)
    assert_close(out[sample], lse[sample], pick(ref[0]), pick(ref[1]), "float16", f"{R} requests")
    if not nested:
        o2, l2 = to_np(*run_gpu(plan, dev, shared=False))
        assert_close(out, lse, o2, l2, "float16", f"{R} requests vs per request")
