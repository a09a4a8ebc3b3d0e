"""Short vectors whose deciding bin, a 128th of an octave, is crowded: light tails, nearly equal or clipped
magnitudes, a layer of like ones. The bin is narrowed and the short lists decide, whatever its size was;
message and residual are the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CHUNK = 1024
REGISTERS, NARROWED = 1, 2


def _values(kind, d, rng, layer=8192):
    sign = rng.choice(np.array([-1.0, 1.0], np.float32), d)
    if kind == "uniform":
        g = rng.uniform(0.0, 1.0, d)
    elif kind == "uniform .55":
        g = rng.uniform(0.0, 0.55, d)
    elif kind == "1 + 5%":
        g = 1.0 + 0.05 * rng.standard_normal(d)
    elif kind == "1 + 1%":
        g = 1.0 + 0.01 * rng.standard_normal(d)
    elif kind == "0.9..1.1":
        g = rng.uniform(0.9, 1.1, d)
    elif kind == "clipped":
        g = np.clip(1.5 * rng.standard_normal(d), -1.0, 1.0) + 1e-3 * rng.standard_normal(d)
    elif kind == "layer":
        g = 1e-2 * rng.standard_normal(d)
        at = d // 2 // (4 * CHUNK) * (4 * CHUNK)
        g[at:at + layer] = rng.uniform(1.0, 1.05, layer)
    elif kind == "normal":
        g = rng.standard_normal(d)
    else:
        g = np.ones(d)
    return (g * sign).astype(np.float32)


def _check(g, r, k, offset=0, force=0, seed=5, step=6):
    from tests import gpu_util as u
    m = np.zeros(len(g), np.float32)
    w = u.GpuWorker(len(g), r, k, residual=m, offset=offset)
    got = w.encode(g, seed, step, force=force)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, seed, step), f"d={len(g)} r={r} k={k}")
    return w.stats["path"], u.lists_that_decided(w.ws)


@pytest.mark.parametrize("kind,d,share", [
    ("uniform", 1 << 21, 0.01), ("uniform", 3_000_017, 0.01), ("uniform .55", 1 << 20, 0.01), ("uniform .55", 1_000_003, 0.05),
    ("1 + 5%", 1 << 20, 0.05), ("1 + 1%", 200_003, 0.01), ("1 + 1%", 3_000_017, 0.005), ("0.9..1.1", 65_536, 0.01),
    ("0.9..1.1", 1 << 20, 0.01), ("clipped", 10_001, 0.1), ("clipped", 200_003, 0.01), ("clipped", 200_003, 0.1),
    ("clipped", 2_097_153, 0.01), ("layer", 65_536, 0.01), ("layer", 200_003, 0.02), ("layer", 250_000, 0.01)])
def test_a_crowded_bin_is_narrowed(kind, d, share):
    g = _values(kind, d, np.random.default_rng(d))
    r = int(d * share)
    for k in (r // (40 if kind == "layer" else 10), r):     # (more of a layer's keys would not fit their list either)
        print(f"narrowed {kind} d={d} r={r} k={k}", flush=True)
        path, how = _check(g, r, k, offset=d % 4)
        assert path == 0 and how & NARROWED, (path, how)


@pytest.mark.parametrize("kind,d,path", [("normal", 200_003, 0), ("normal", 2_097_152, 0), ("signs", 200_003, 4), ("signs", 2_097_152, 4)])
def test_others_are_not(kind, d, path):
    """Few entries; equal ones, of which no part is smaller."""
    g = _values(kind, d, np.random.default_rng(d))
    got, how = _check(g, d // 100, d // 1000)
    assert got == path and how & NARROWED == 0, (got, how)


@pytest.mark.parametrize("layer,count,narrowed", [(4096, 383, False), (4096, 384, False), (4096, 385, True), (4096, 1000, True),
                                                  (1024, 383, False), (1024, 385, True)])
def test_entries_in_one_workgroups_chunks(layer, count, narrowed):
    """`count` entries of the deciding bin within `layer` elements: the list of one workgroup holds 384, and where a
    workgroup has more the bin counts as crowded, few as its entries are."""
    d = 300_000
    rng = np.random.default_rng(layer + count)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    g[rng.permutation(d)[:900]] = (rng.standard_normal(900) + 30.0).astype(np.float32)
    at = 100 * CHUNK + rng.permutation(layer)[:count]
    g[at] = (1.0 + rng.permutation(1 << 15)[:count] / 2.0 ** 23).astype(np.float32)
    r = int((np.abs(g) > 0.5).sum()) - count // 2
    for k in (r // 4, r):
        path, how = _check(g, r, k)
        assert path == 0 and bool(how & NARROWED) == narrowed, (path, how)


@pytest.mark.parametrize("low", [0, 255])
@pytest.mark.parametrize("take", [1, 2, 1599, 1600])
def test_the_first_and_last_part(low, take):
    """All entries of the deciding bin in its lowest or highest part, and the cut at either end of them."""
    d = 50_000
    rng = np.random.default_rng(low + take)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    at = rng.permutation(d)
    g[at[:300]] = (rng.standard_normal(300) + 30.0).astype(np.float32)
    pattern = (0x3F800000 | low << 8) + rng.integers(0, 256, 1600)
    g[at[300:1900]] = pattern.astype(np.uint32).view(np.float32)
    r = 300 + take
    path, how = _check(g, r, r // 3)
    assert path & 3 == 0 and how & NARROWED, (path, how)


@pytest.mark.parametrize("force", ["CHECK_IN_ABORT", "KEY_WINDOW_MISS", "ESTIMATE_MISS"])
@pytest.mark.parametrize("kind,d", [("1 + 1%", 12_000), ("clipped", 60_000), ("uniform", 1 << 21), ("layer", 300_000)])
def test_crowded_bins_and_forced_fallbacks(kind, d, force):
    """Nobody narrows; the key cut from a selection over all candidates; the vector itself walked."""
    import paper_2005_10761_amd as rt
    g = _values(kind, d, np.random.default_rng(d))
    r = d // 100
    path, how = _check(g, r, r // 3, offset=1, force=getattr(rt, "FORCE_" + force))
    assert how & NARROWED == 0 if force != "KEY_WINDOW_MISS" else path & 1, (path, how)


# every classify workgroup picks; a kernel does
@pytest.mark.parametrize("n,d", [(3, 500_000), (8, 200_003), (3, 2_097_152), (16, 1 << 20)])
def test_batches_that_narrow(n, d):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    r, k = d // 100, d // 1000
    kinds = ("uniform .55", "clipped", "normal")
    gs = [_values(kind, d, np.random.default_rng(d + i)) for i, kind in enumerate(kinds)]
    dev = [torch.from_numpy(g).to(u.DEV) for g in gs]
    res = [torch.zeros(d, device=u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    print(f"narrowed batch n={n} d={d}", flush=True)
    rt.encode_batch([dev[w % 3] for w in range(n)], res, r, k, list(range(n)), 3, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        st = rt.encode_stats(ws[w * stride:(w + 1) * stride])
        assert st["path"] == 0 and st["error_flags"] == 0, (w, st)
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        if w < 3:
            u.assert_encode_equal(got, oracle.encode(gs[w], np.zeros(d, np.float32), r, k, w, 3), f"member {w} of {n}")


def test_three_streams_that_narrow_at_once():
    """Each grid waits for its own workgroups; one that cannot have them all goes on without narrowing."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    n, d = 3, 3_000_000
    r, k = d // 100, d // 1000
    gs = [_values("1 + 1%", d, np.random.default_rng(w)) for w in range(n)]
    ms = [np.zeros(d, np.float32) for _ in range(n)]
    streams = [torch.cuda.Stream(device=u.DEV) for _ in range(n)]
    dev = [torch.from_numpy(g).to(u.DEV) for g in gs]
    res = [torch.zeros(d, device=u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    ws = [torch.empty(rt.encode_workspace_bytes(d, r, k), dtype=torch.uint8, device=u.DEV) for _ in range(n)]
    torch.cuda.synchronize()
    for t in range(2):
        for w in range(n):
            rt.encode(dev[w], res[w], r, k, 7 + w, t, idx[w], val[w], ws[w], stream=streams[w])
        torch.cuda.synchronize()
        for w in range(n):
            assert rt.encode_stats(ws[w])["error_flags"] == 0
            want = oracle.encode(gs[w], ms[w], r, k, 7 + w, t)
            got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
            u.assert_encode_equal(got, want, f"step {t} stream {w}")
            ms[w] = want[2]


def test_narrowing_in_a_captured_graph():
    """The counters that the workgroups share are cleared by every replay."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    d = 400_000
    r, k = d // 100, d // 1000
    gs = [_values(kind, d, np.random.default_rng(i)) for i, kind in enumerate(("clipped", "uniform", "1 + 1%", "normal"))]
    w = u.GpuWorker(d, r, k)
    w.grad.copy_(torch.from_numpy(gs[0]))
    stream = torch.cuda.Stream(device=u.DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        rt.encode(w.grad, w.residual, r, k, 9, 2, w.idx, w.val, w.ws, stream=torch.cuda.current_stream())
    for g in gs + gs[:1]:
        w.grad.copy_(torch.from_numpy(g))
        w.residual.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = (w.idx.cpu().numpy().view(np.uint32), w.val.cpu().numpy(), w.residual.cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, np.zeros(d, np.float32), r, k, 9, 2), "replay")
        assert rt.encode_stats(w.ws)["path"] == 0
        u.gpu_encode_once(gs[1], np.zeros(d, np.float32), r, k, 1, 1)      # eager work between the replays
