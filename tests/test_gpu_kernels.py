"""GPU kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest

import coe_workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_02354_amd import binding
    return binding


@pytest.mark.parametrize("n,E", [(1, 2048), (63, 511), (64, 512), (65, 513), (511, 1), (2047, 370), (2048, 370), (2049, 370),
                                 (4097, 2048), (100003, 370), (262144, 33), (262145, 33), (300001, 600)])
def test_regroup_range_edges(B, oracle, n, E):
    """One workgroup up to 2048 keys, then ranges of 2048, then longer ranges beyond 128 workgroups."""
    rng = np.random.default_rng(n + E)
    cur = np.where(rng.random(n) < 0.8, rng.choice(E, size=n, p=W.zipf_probs(E, 1.1)), rng.choice([-1, E, E + 5], size=n)).astype(np.int32)
    ctx = B.Context(max_requests=n)
    got = ctx.coe_debug_regroup(cur, E)
    ctx.close()
    want = oracle.regroup(np.where(cur < E, cur, -1).astype(np.int32), E)
    for k in ("cnt", "off", "perm", "inv"):
        assert np.array_equal(got[k], want[k]), k
