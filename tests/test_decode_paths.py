"""Which path a decode call of given sizes takes (CPU: the choice reads host
scalars only; 256 compute units are assumed without a GPU): one launch for small
calls, two kernels where the bytes, unbalanced contexts or prefixes without
further readers make the one launch the slower one.  The figures are measured on
MI355X, two kernels / one launch, in microseconds."""
import ctypes

import pytest

from paper_2405_19888_amd import binding as B


def waves(lib, requests, heads, groups=0, prefix=0, own=16, per_request=False, dtype=1, head_dim=128, readers=None,
          depth=0):
    prob = B.make_problem(
        num_requests=requests, num_heads=heads, head_dim=head_dim, block_size=16, num_groups=groups,
        max_group_size=readers or -(-requests // groups) if groups else 0, max_prefix_len=prefix if groups else 0,
        max_suffix_len=own, prefix_table_stride=-(-prefix // 16), suffix_table_stride=-(-own // 16),
        num_prefix_blocks=65536, num_suffix_blocks=65536, dtype=dtype, sm_scale=0.1, max_prefix_depth=depth)
    return lib.parrot_test_decode_waves(ctypes.byref(prob), int(per_request))


@pytest.mark.parametrize("kw", [
    dict(requests=29, heads=40, groups=22, prefix=1062, own=882),                  # 131 / 177
    dict(requests=39, heads=8, groups=20, prefix=2000, own=1240),                  # 47 / 62
    dict(requests=4, heads=32, groups=3, prefix=3000, own=60),                     # 35.7 / 46.1
    dict(requests=4, heads=32, groups=120, prefix=3000, own=60, readers=2),        # 37.8 / 45.9, most groups unread
    dict(requests=16, heads=8, groups=11, prefix=3583, own=1793),                  # 46 / 67
    dict(requests=9, heads=16, groups=3, prefix=2048, own=1401),                   # 28 / 42
    dict(requests=9, heads=40, groups=8, prefix=1958, own=391, per_request=True),  # 29.9 / 51
    dict(requests=8, heads=32, own=1000),                                          # 28.6 / 29.6
    dict(requests=32, heads=32, own=300),                                          # 33.1 / 40.0
    dict(requests=4, heads=32, own=4000),                                          # 27.8 / 45.8
    dict(requests=8, heads=32, own=4097),                                          # past a lane's table entries
])
def test_calls_kept_on_two_kernels(parrot_lib, kw):
    assert waves(parrot_lib, **kw) == 0


@pytest.mark.parametrize("kw,n", [
    (dict(requests=4, heads=4, groups=1, prefix=128, own=32, dtype=0, head_dim=64), 8),   # 9.4 / 4.4
    (dict(requests=7, heads=32, groups=1, prefix=317, own=700, readers=4), 8),            # 17.5 / 11.4
    (dict(requests=8, heads=32, own=300), 8),                                             # 15.3 / 10.8
    (dict(requests=8, heads=32, groups=1, prefix=500, own=50), 8),                        # 10.9 / 9.3
    (dict(requests=8, heads=32, groups=1, prefix=500, own=50, per_request=True), 8),      # 12.9 / 9.3
    (dict(requests=32, heads=32, own=50), 4),                                             # 14.2 / 9.6
    (dict(requests=2, heads=8, groups=2, prefix=64, own=40, depth=2), 8),
])
def test_small_calls_take_one_launch(parrot_lib, kw, n):
    assert waves(parrot_lib, **kw) == n


def test_forced_paths(parrot_lib):
    small, large = dict(requests=4, heads=4, own=32), dict(requests=32, heads=32, own=300)
    try:
        parrot_lib.parrot_test_decode_path(0)
        assert waves(parrot_lib, **small) == 0
        parrot_lib.parrot_test_decode_path(1)
        assert waves(parrot_lib, **large) == 4
        assert waves(parrot_lib, requests=2, heads=2, own=4097) == 0      # its lists do not fit
        assert waves(parrot_lib, requests=1 << 17, heads=32, own=16) == 4
        assert waves(parrot_lib, requests=1 << 18, heads=32, own=16) == 0  # nor one launch (2^32 threads)
        parrot_lib.parrot_test_decode_path(8)
        assert waves(parrot_lib, **large) == 8
    finally:
        parrot_lib.parrot_test_decode_path(-1)
    assert waves(parrot_lib, **small) == 8 and waves(parrot_lib, **large) == 0
