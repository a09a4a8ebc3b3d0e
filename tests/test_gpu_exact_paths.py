"""The exact selections behind the key window, the bracket and the short lists:
which members the streaming kernel left out decides whether its candidate buffer
will do or has to be completed from the vector first. Against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SEED, STEP = 21, 6


def _smallest_keys(d, count):
    """The coordinates with the smallest sampling keys: what random-k sends."""
    zero = np.zeros(d, np.float32)
    return oracle.encode(zero, zero, d, count, SEED, STEP)[0]


def _inputs(kind, d, r, rng):
    g = rng.standard_normal(d).astype(np.float32) * np.float32(1e-3)
    if kind in ("low", "high"):       # the top r are the coordinates with the smallest (largest) keys of all
        chosen = np.zeros(d, bool)
        chosen[_smallest_keys(d, r if kind == "low" else d - r)] = True
        g[chosen == (kind == "low")] *= np.float32(1e5)
    elif kind == "crowded":           # the top r are neighbours: the key list of one workgroup overflows
        g[d // 2: d // 2 + r] *= np.float32(1e5)
    return g, np.zeros(d, np.float32)


@pytest.mark.parametrize("abort", [False, True])
@pytest.mark.parametrize("d,r,k", [(70_001, 3_000, 1_500), (300_001, 3_000, 1_500), (5_000_011, 50_000, 25_000)])
@pytest.mark.parametrize("kind", ["low", "high", "crowded", "window", "bracket"])
def test_exact_selections(kind, d, r, k, abort):
    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    force = {"window": rt.FORCE_KEY_WINDOW_MISS, "bracket": rt.FORCE_BRACKET_LOW}.get(kind, 0)
    force |= rt.FORCE_CHECK_IN_ABORT if abort else 0
    print(f"exact selection: {kind} d={d} r={r} k={k} abort={abort}", flush=True)
    g, m = _inputs(kind, d, r, np.random.default_rng(d))
    got = u.gpu_encode_once(g, m, r, k, SEED, STEP, offset=d % 4, force=force)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, SEED, STEP), f"{kind} d={d}")
    st = got[3]
    # exact, and not by walking the vector pass after pass (a short vector's candidates are all
    # there: with few of them above a bracket that is too low the short lists still decide)
    assert st["path"] & 3 == 1 or (kind == "bracket" and d < 1 << 21 and st["path"] == 0), st
    if d > 1 << 22 and kind in ("high", "window", "bracket"):
        # members whose keys lie above the window decide: the buffer was completed with them.
        # (The bracket of 65,536 samples holds 0.7 r entries; what is above it and not to be sent
        # had been left out.)
        assert st["superset_size"] >= r, st
