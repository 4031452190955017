"""A workgroup's tile without a division (scc_common.h, dealt): the reciprocal's quotient and its one correction are exact."""
import numpy as np
import pytest


@pytest.mark.parametrize("inner", [1, 2, 3, 7, 12, 255, 256, 257, 1000, 65535, 65536, 65537, 2**30, 2**31 - 1])
def test_quotient_is_exact(inner):
    recip = 2**32 - 1 if inner == 1 else 2**32 // inner          # make_runs
    some = np.random.default_rng(0).integers(0, 2**31, 20000)
    ends = np.arange(1, 2000, dtype=np.int64) * inner
    at = np.concatenate([np.arange(2000), some, ends, ends - 1, [2**31 - 1]])
    at = at[at < 2**31]
    tile = (at.astype(np.uint64) * np.uint64(recip) >> np.uint64(32)).astype(np.int64)
    rest = at - tile * inner
    more = rest >= inner
    assert np.array_equal(tile + more, at // inner) and np.array_equal(rest - more * inner, at % inner)
