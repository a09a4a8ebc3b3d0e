"""Short vectors, whose magnitudes are all counted by their leading 15 bits while they are added:
lengths on both sides of every change of launch shape, octaves that meet in one slot of a
workgroup's row, a cut among zeros and denormals. Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CHUNK = 1024


def _check(g, m, r, k, seed=5, step=6, offset=0, path=0, force=0):
    from tests import gpu_util as u
    got = u.gpu_encode_once(g, m, r, k, seed, step, offset=offset, force=force)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, seed, step), f"d={len(g)} r={r} k={k}")
    if path is not None:
        assert got[3]["path"] == path, got[3]
    return got[3]


# 8 and 16 wavefronts per workgroup, a second round of chunks, the last counted length
@pytest.mark.parametrize("chunks", [1, 7, 8, 9, 512, 513, 2047, 2048, 2049, 2064, 3071, 3072, 3073])
@pytest.mark.parametrize("ragged", [0, 513])
@pytest.mark.parametrize("of_r", ["sparse", "dense", "top-k"])
def test_lengths(chunks, ragged, of_r):
    d = (chunks - 1) * CHUNK + (ragged or CHUNK)
    rng = np.random.default_rng(chunks * 3 + ragged)
    g = (rng.standard_normal(d) * 10.0 ** rng.uniform(-3, 0, d)).astype(np.float32)
    m = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    r = min(d, max(2, d // (5 if of_r == "dense" else 90)))
    k = r if of_r == "top-k" else max(1, r // 6)
    print(f"counted chunks={chunks} ragged={ragged} r={r} k={k}", flush=True)
    _check(g, m, r, k, offset=(chunks + ragged) % 4, path=None if chunks < 10 else 0)


@pytest.mark.parametrize("d,r", [(2500 * CHUNK, 1 << 15), (2500 * CHUNK, (1 << 15) + 1), (2048 * CHUNK, 1 << 16),
                                 (2048 * CHUNK, (1 << 16) + 1), (1024 * CHUNK, 1 << 18), (1025 * CHUNK, 1 << 18),
                                 (1 << 18, (1 << 18) - 1)])
def test_large_top_sets(d, r):
    rng = np.random.default_rng(r)
    g = rng.standard_normal(d).astype(np.float32)
    _check(g, np.zeros(d, np.float32), r, r // 20, path=None)


# rows of all members up to 256: every classify workgroup picks; beyond: a kernel
@pytest.mark.parametrize("n,chunks", [(16, 128), (16, 129), (2, 2048), (3, 2048), (17, 100), (7, 2500)])
def test_batches(n, chunks):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    d = chunks * CHUNK - 3
    r, k = d // 50, d // 500
    rng = np.random.default_rng(n + chunks)
    gs = [(rng.standard_normal(d) * 10.0 ** rng.uniform(-3, 0, d)).astype(np.float32) for _ in range(2)]
    m = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    dev = [torch.from_numpy(g).to(u.DEV) for g in gs]
    res = [torch.from_numpy(m).to(u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    print(f"counted batch n={n} chunks={chunks}", flush=True)
    rt.encode_batch([dev[w % 2] for w in range(n)], res, r, k, list(range(n)), 3, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        st = rt.encode_stats(ws[w * stride:(w + 1) * stride])
        assert st["path"] == 0 and st["error_flags"] == 0, (w, st)
        if w in (0, 1, n - 1):
            got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
            u.assert_encode_equal(got, oracle.encode(gs[w % 2], m, r, k, w, 3), f"member {w} of {n}")


# the cut among the large ones; among those that lost their slot (their octave is narrowed; unless nobody narrows)
@pytest.mark.parametrize("d", [40_000, 300_007, 2_097_152])
@pytest.mark.parametrize("r,force,path", [(100, 0, 0), (5_000, 0, 0), (5_000, "CHECK_IN_ABORT", 2)])
def test_octaves_that_meet_in_a_slot(d, r, force, path):
    """A few hundred elements around 2^40, all others 64 octaves below: their bins share a slot of the rows."""
    import paper_2005_10761_amd as rt
    r = max(r, d // 50) if r != 100 else r
    rng = np.random.default_rng(d + r)
    g = (rng.uniform(1.0, 2.0, d) * 2.0 ** -24).astype(np.float32)
    g[::97] = (rng.uniform(1.0, 2.0, len(g[::97])) * 2.0 ** 40).astype(np.float32)
    g *= rng.choice(np.array([-1.0, 1.0], np.float32), d)
    st = _check(g, np.zeros(d, np.float32), r, r // 10, path=None, force=getattr(rt, f"FORCE_{force}") if force else 0)
    assert st["path"] == 0 if path == 0 else st["path"] & 2, st


@pytest.mark.parametrize("d", [2, 3, 4, 5, 63, 257, 1025])
@pytest.mark.parametrize("top", [np.inf, np.nan, 2.0 ** 64])
def test_octaves_that_meet_in_tiny_vectors(d, top):
    """The smallest vectors whose deciding octave lost its slot: to infinities, to what is no number, to one value."""
    rng = np.random.default_rng(d)
    g = rng.uniform(1.0, 2.0, d).astype(np.float32)
    g[rng.integers(0, d)] = top
    for r in {2, d // 2 + 1, d - 1}:
        if 2 <= r < d:
            print(f"tiny d={d} r={r} top={top}", flush=True)
            _check(g, np.zeros(d, np.float32), r, (r + 1) // 2, path=None)
            _check(g, np.zeros(d, np.float32), r, r, offset=1, path=None)


@pytest.mark.parametrize("n,abort", [(3, False), (16, False), (16, True)])      # every classify workgroup picks; a kernel does, and nobody narrows
def test_denormals_below_an_octave_that_shares_their_slot(n, abort):
    """The octave of the denormals, zeros among them, is the one that lost its slot."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    d = 200_000
    rng = np.random.default_rng(n)
    g = (rng.integers(0, 1 << 23, d) * (rng.random(d) < 0.7)).astype(np.uint32)
    g[::97] = (rng.integers(0, 1 << 23, len(g[::97])) | 64 << 23).astype(np.uint32)
    g = g.view(np.float32)
    r, k = d // 2, d // 20
    grad = torch.from_numpy(g).to(u.DEV)
    res = [torch.zeros(d, device=u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    if abort:
        rt.force_next_encode(rt.FORCE_CHECK_IN_ABORT)
    rt.encode_batch([grad] * n, res, r, k, list(range(n)), 3, idx, val, ws)
    torch.cuda.synchronize()
    for w in (0, n - 1):
        st = rt.encode_stats(ws[w * stride:(w + 1) * stride])
        assert (st["path"] & 2 if abort else st["path"] == 0) and st["error_flags"] == 0, (w, st)
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, np.zeros(d, np.float32), r, k, w, 3), f"member {w} of {n}")


@pytest.mark.parametrize("d", [5_000, 300_007, 2_500_000])
@pytest.mark.parametrize("kind", ["zeros decide", "all zero", "denormals", "smallest denormals", "specials", "octaves"])
def test_where_the_cut_may_lie(d, kind):
    rng = np.random.default_rng(d)
    r, k = d // 10, d // 30
    g = np.zeros(d, np.float32)
    some = rng.permutation(d)
    if kind == "zeros decide":
        g[some[:r // 2]] = rng.standard_normal(r // 2).astype(np.float32)
        g[some[r // 2:r]] = np.float32(-0.0)
    elif kind == "denormals":                       # bins 1 to 127: the group of exponent zero
        g = (rng.integers(1, 1 << 23, d).astype(np.uint32) | (rng.integers(0, 2, d).astype(np.uint32) << 31)).view(np.float32)
    elif kind == "smallest denormals":              # bin 0 holds distinct magnitudes
        g = rng.integers(0, 1 << 16, d).astype(np.uint32).view(np.float32)
    elif kind == "specials":
        g = rng.standard_normal(d).astype(np.float32)
        g[some[:20]] = np.float32("inf")
        g[some[20:30]] = np.float32("-inf")
        g[some[30:40]] = np.float32("nan")
    elif kind == "octaves":                         # every binade there is
        g = (rng.integers(0, 255 << 23, d).astype(np.uint32)).view(np.float32)
    print(f"cut {kind} d={d}", flush=True)
    _check(g, np.zeros(d, np.float32), r, k, offset=1, path=None)
    _check(g, np.zeros(d, np.float32), r, r, path=None)


@pytest.mark.parametrize("count", [127, 128, 129, 1024])
@pytest.mark.parametrize("d", [100_000, 2_600_000])             # all members stay in the buffer; those that may be sent
def test_chunks_that_fill_their_slice(d, count):
    rng = np.random.default_rng(d + count)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    for c0 in (0, 5 * CHUNK, d // CHUNK * CHUNK - CHUNK):
        g[c0 + rng.permutation(CHUNK)[:count]] = (rng.standard_normal(count) + 30.0).astype(np.float32)
    for r, k in ((3 * count + 500, 300), (3 * count + 500, 3 * count + 500)):
        _check(g, np.zeros(d, np.float32), r, k, path=None)


# 25, 123 and 256 classify workgroups, of which 256, 64 and 32 places per list fit registers (8 fetched at once)
@pytest.mark.parametrize("d", [100_003, 500_000, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("hot", [9, 40, 70, 290])
@pytest.mark.parametrize("where", ["window", "bin", "few levels"])
def test_lists_in_and_beyond_registers(d, hot, where):
    """`hot` members in one classify workgroup's chunks: nearly half of their keys lie in the window; or they
    share the deciding bin, with the cut among them, as distinct magnitudes or as three. Few of them are found in
    registers where there are at most 256 such workgroups; 290 entries of the bin are in no register, but in a list."""
    from tests import gpu_util as u
    rng = np.random.default_rng(d + hot)
    g = (rng.standard_normal(d) * 1e-6).astype(np.float32)
    g[rng.permutation(d)[:200]] = (rng.standard_normal(200) + 9.0).astype(np.float32)
    at = 8 * CHUNK + rng.permutation(4 * CHUNK)[:hot]
    if where == "window":
        g[at] = (rng.standard_normal(hot) + 9.0).astype(np.float32)
    elif where == "bin":
        g[at] = (1.0 + rng.permutation(1 << 15)[:hot] / 2.0 ** 23).astype(np.float32)
    else:
        g[at] = (1.0 + rng.integers(0, 3, hot) / 2.0 ** 20).astype(np.float32)
    r = len(np.flatnonzero(np.abs(g) > 0.5)) - (0 if where == "window" else hot // 2)
    print(f"lists d={d} hot={hot} {where} r={r}", flush=True)
    for k in (r // 3, r):
        w = u.GpuWorker(d, r, k, residual=np.zeros(d, np.float32))
        got = w.encode(g, 5, 6)
        u.assert_encode_equal(got, oracle.encode(g, np.zeros(d, np.float32), r, k, 5, 6), f"d={d} r={r} k={k}")
        decided = w.stats["path"], u.lists_that_decided(w.ws)
        if hot == 9:
            assert decided == (0, 1 if d <= 1 << 20 else 0), decided
        elif hot == 290 and where != "window":
            assert decided == (0, 0), decided


@pytest.mark.parametrize("d", [5_000, 300_007, 2_500_000])
def test_a_forced_miss_runs_the_counted_chain(d):
    """What the hook makes happen, happens on the kernels such a vector takes: no estimate has left its bins behind."""
    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    g = np.random.default_rng(d).standard_normal(d).astype(np.float32)
    w = u.GpuWorker(d, d // 100, d // 500)
    want = oracle.encode(g, np.zeros(d, np.float32), d // 100, d // 500, 1, 2)
    u.assert_encode_equal(w.encode(g, 1, 2, force=rt.FORCE_ESTIMATE_MISS), want, f"d={d}")
    assert w.stats["path"] & 3 == 3 and u.estimated_bins(w.ws) == 0
