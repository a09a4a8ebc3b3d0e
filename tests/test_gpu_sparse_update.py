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


def _own_region(rng, k):   # one of eight stretches of the vector
    return rng.integers(8) * (D // 8) + np.sort(rng.choice(D // 8, k, replace=False))


def _repeats(rng, k):      # an index that fills more than one window of 256, others twice
    a = np.repeat(np.sort(rng.choice(D, k // 2 + 1, replace=False)), 2)[:k]
    a[k // 3: k // 3 + min(700, k // 2)] = a[k // 3]
    return np.sort(a)


def _runs(rng, k):         # runs around a wavefront's 64 and a window's 256 entries, and one that fills several windows
    lengths = np.tile([1, 2, 63, 64, 65, 1, 255, 256, 257, 3, 513, 900], k // 2180 + 1)
    starts = np.sort(rng.choice(D, len(lengths), replace=False))
    return np.repeat(starts, lengths)[:k]


@pytest.mark.parametrize("n,k", [(1, 1), (1, 255), (1, 256), (1, 257), (2, 1000), (3, 255), (4, 512),
                                 (5, 4687), (8, 24576), (8, 64)])
@pytest.mark.parametrize("layout", [_spread, _packed, _ends, _own_region, _repeats, _runs])
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


PIECE = 1 << 28              # (torch has no arange, fill or comparison of 2^32 elements)


def _weights(d):
    import torch
    from tests import gpu_util as u
    w = torch.empty(d, device=u.DEV)
    for i in range(0, d, PIECE):
        torch.arange(min(PIECE, d - i), out=w[i:i + PIECE])
    return w


VALUES = np.array([2.0**24, 1.0, -2.0**24, 0.5, -0.0, 1e-45, 3e-39], np.float32)


@pytest.mark.parametrize("d", [1 << 25, (1 << 25) - 1, (1 << 26) + 77, (1 << 28) + 1, (1 << 32) - 1])
@pytest.mark.parametrize("n", [1, 8, 9])
@pytest.mark.parametrize("specials", [False, True])
def test_sparse_update_over_the_rule(d, n, specials):
    """Lengths and worker counts on both sides of the rule, up to the longest vector;
    infinities and not-a-numbers among values and weights. A coordinate's new weight
    depends on its own entries alone: the oracle runs on the coordinates that were sent,
    renumbered, and every other weight must keep its bits."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    k = 3000
    print(f"sparse update d={d} n={n} specials={specials}", flush=True)
    rng = np.random.default_rng(d % 1000 + n)
    hot = rng.integers(0, d, 400)                  # coordinates that several workers send
    idx = [np.unique(np.concatenate((rng.integers(0, d, 2 * k), hot[rng.random(400) < 0.5], [0, d - 1])))
           for _ in range(n)]
    idx = np.concatenate([np.sort(rng.permutation(i[1:-1])[:k - 2].tolist() + [0, d - 1]) for i in idx]).astype(np.int64)
    values = np.append(VALUES, [np.inf, -np.inf, np.nan, 3.4e38]).astype(np.float32) if specials else VALUES
    val = rng.choice(values, n * k)
    sent, place = np.unique(idx, return_inverse=True)
    at = torch.from_numpy(sent).to(u.DEV)
    omega = _weights(d)
    if specials:
        omega[at[::5]] = float("inf")
        omega[at[::7]] = float("nan")
    before = omega[at].cpu().numpy()
    want = oracle.aggregate_update_f32(place.astype(np.uint32), val, n, len(sent), 0.37, 3.0, before)
    ti = torch.from_numpy(idx.astype(np.uint32).view(np.int32)).to(u.DEV)
    tv = torch.from_numpy(val).to(u.DEV)
    ws = torch.empty(rt.aggregate_update_workspace_bytes(d, n, k), dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.aggregate_update(ti, tv, n, k, 0.37, 3.0, omega, ws)
    assert u.same_floats(omega[at].cpu().numpy(), want)
    omega[at] = 0.0
    rest = _weights(d)
    rest[at] = 0.0
    for i in range(0, d, PIECE):
        assert torch.equal(omega[i:i + PIECE], rest[i:i + PIECE]), i
