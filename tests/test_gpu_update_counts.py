"""The sparse weight step of long vectors with few entries, whose workgroups first learn how many entries
they have: totals on both sides of every change of grid and kernel, ranges that hold more than the
hash table takes, coordinates sent by several workers, repeated indices. Bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

D = (1 << 25) + 5


@pytest.mark.parametrize("entries", [8, 8192, 8200, 1 << 17, (1 << 17) + 8])
@pytest.mark.parametrize("n", [1, 8])
@pytest.mark.parametrize("layout", ["crowded", "same", "repeats", "ends"])
def test_totals_and_layouts(entries, n, layout):
    from tests import gpu_util as u
    k = max(1, entries // n)
    rng = np.random.default_rng(entries + n)
    if layout == "crowded":                          # half of every message spread out, half in a stretch of its own length
        def one():
            a = rng.choice(D, k, replace=False)
            at = int(rng.integers(0, D - k))
            a[:k // 2] = at + np.arange(k // 2)
            return np.sort(a)
        idx = np.stack([one() for _ in range(n)])
    elif layout == "same":                           # all workers send the same coordinates
        idx = np.stack([np.sort(rng.choice(D, k, replace=False))] * n)
    elif layout == "repeats":
        idx = np.sort(rng.integers(0, max(2, min(D, k * 3)), (n, k)), axis=1)
        idx[:, :k // 8] = idx[:, k // 8:k // 8 + 1]  # a long run of one coordinate
        idx = np.sort(idx, axis=1)
    else:                                            # both ends of the vector
        idx = np.sort(np.concatenate([np.tile(np.arange(k // 2), (n, 1)), np.tile(D - 1 - np.arange(k - k // 2), (n, 1))], axis=1), axis=1)
    idx = idx.astype(np.uint32)
    val = rng.standard_normal((n, k)).astype(np.float32)
    val[0, :2] = [np.float32("inf"), np.float32(-0.0)][:min(2, k)]
    omega = rng.standard_normal(D, dtype=np.float32)
    print(f"update counts entries={entries} n={n} {layout}", flush=True)
    got = u.gpu_aggregate_update(idx, val, n, D, 0.1, 1.5, omega, offset=1)
    want = oracle.aggregate_update_f32(idx, val, n, D, 0.1, 1.5, omega)
    assert u.same_floats(got, want)
