"""The sparse weight step on sparse messages (the kernel that sums in a hash
table): bit for bit against the oracle's binary32 worker-order variant."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# from 2^25 coordinates on, up to 8 workers and 12 entries per 2048 coordinates go through the hash kernel
D = (1 << 25) + 3


def _spread(rng, k):
    return np.sort(rng.choice(D, k, replace=False))


def _packed(rng, k):       # neighbouring coordinates: the same table slots probed, many rounds of 256
    return np.arange(k) + rng.integers(1000, 1100)


def _ends(rng, k):         # the first and the last coordinates of the vector
    return np.concatenate((np.arange(k // 2), np.arange(D - (k - k // 2), D)))


def _own_region(rng, k, w=[0]):
    w[0] += 1
    return (w[0] % 8) * (D // 8) + np.sort(rng.choice(D // 8, k, replace=False))


def _repeats(rng, k):      # an index that fills more than one window of 256, others twice
    a = np.repeat(np.sort(rng.choice(D, k // 2 + 1, replace=False)), 2)[:k]
    a[k // 3: k // 3 + min(700, k // 2)] = a[k // 3]
    return np.sort(a)


@pytest.mark.parametrize("n,k", [(1, 1), (1, 255), (1, 256), (1, 257), (2, 1000), (3, 255), (4, 512),
                                 (5, 4687), (8, 24576), (8, 64)])
@pytest.mark.parametrize("layout", [_spread, _packed, _ends, _own_region, _repeats])
def test_sparse_update_matches_the_oracle(n, k, layout):
    from tests import gpu_util as u
    rng = np.random.default_rng(1000 * n + k)
    idx = np.concatenate([layout(rng, k) for _ in range(n)]).astype(np.uint32)
    # few distinct values: sums cancel to zero, and their order shows (2^24, 1, -2^24)
    val = rng.choice(np.array([2.0**24, 1.0, -2.0**24, 0.5, -0.0, 1e-45, 3e-39], np.float32), n * k)
    omega = np.tile(rng.standard_normal(4096).astype(np.float32), D // 4096 + 1)[:D]
    eta, scale = ((0.1, 1.0), (-0.37, 5.0))[k % 2]
    got = u.gpu_aggregate_update(idx, val, n, D, eta, scale, omega, offset=n % 2)
    want = oracle.aggregate_update_f32(idx, val, n, D, eta, scale, omega)
    assert np.array_equal(u.bits(got), u.bits(want))
