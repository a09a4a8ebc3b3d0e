"""The streaming kernel's launch shapes and the candidates it leaves out: chunk
counts on both sides of each change of shape, gradient and residual at
different 4-byte offsets, layers so hot that most candidates lie above the
bracket (and are dropped unless they may be sent), against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,off_g,off_m", [
    (1024, 0, 0), (1023, 1, 2), (1025, 3, 0),
    (1024 * 1024, 0, 1), (1024 * 1024 + 1, 0, 0),            # one more chunk than 4 wavefronts x 256
    (2048 * 1024, 2, 0), (2048 * 1024 + 257, 0, 3),          # the last length with two rows at a time
    ((1 << 24) - 1, 0, 0), ((1 << 24) + 5, 1, 1),            # 12 and 10 wavefronts per workgroup
    # what the last chunk holds, around whole groups of one row and of two
    (5120 + 255, 0, 0), (5120 + 511, 0, 1), (5120 + 512, 1, 0), (5120 + 513, 0, 0), (5120 + 1023, 2, 2),
    (2099 * 1024 + 255, 0, 0), (2099 * 1024 + 256, 0, 0), (2099 * 1024 + 511, 3, 1), (2099 * 1024 + 512, 0, 0),
    (2099 * 1024 + 1023, 0, 2), ((1 << 25) + 1700, 1, 0),
])
@pytest.mark.parametrize("layout", ["even", "hot"])
def test_stream_shapes(d, off_g, off_m, layout):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    rng = np.random.default_rng(d + off_g)
    g = rng.standard_normal(d).astype(np.float32)
    if layout == "hot":
        g *= np.float32(1e-3)
        g[d // 3: d // 3 + max(1, d // 50)] *= np.float32(1e4)
    m = (rng.standard_normal(d) * 1e-4).astype(np.float32)
    for r, k in ((max(1, d // 60), max(1, d // 600)), (max(1, d // 100), max(1, d // 100)), (d, max(1, d // 100))):
        tg = torch.zeros(d + off_g, device=u.DEV)[off_g:]
        tm = torch.zeros(d + off_m, device=u.DEV)[off_m:]
        tg.copy_(torch.from_numpy(g))
        tm.copy_(torch.from_numpy(m))
        idx = torch.empty(k, dtype=torch.int32, device=u.DEV)
        val = torch.empty(k, device=u.DEV)
        ws = torch.empty(rt.encode_workspace_bytes(d, r, k), dtype=torch.uint8, device=u.DEV)
        ws.fill_(0xA5)
        rt.encode(tg, tm, r, k, 3, 4, idx, val, ws)
        st = rt.encode_stats(ws)
        # (a layer of few chunks puts more keys of the window than its 128 places into one
        # classify workgroup's list: the exact selection then decides, as it does by design)
        assert st["error_flags"] == 0 and (layout == "hot" or st["path"] == 0), st
        got = (idx.cpu().numpy().view(np.uint32), val.cpu().numpy(), tm.cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, m, r, k, 3, 4), f"d={d} r={r} k={k}")


@pytest.mark.parametrize("chunks,whole", [(2048, True), (2049, False), (3072, False), (3073, True), (4096, True),
                                          (4097, False)])
@pytest.mark.parametrize("ops", ["rtopk", "top-k", "random-k"])
def test_short_vectors_keep_every_candidate(chunks, whole, ops):
    """Part of the top r lies far above the bracket: a keying stream leaves out what will not
    be sent of it, a short vector's keeps all candidates."""
    from tests import gpu_util as u
    d = chunks * 1024 - 5
    rng = np.random.default_rng(chunks)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    g[::50] *= np.float32(1e4)
    g[::400] *= np.float32(1e4)              # a quarter of the top r, far above the rest
    m = np.zeros(d, np.float32)
    r = d if ops == "random-k" else d // 100
    k = r if ops == "top-k" else d // 1000
    got = u.gpu_encode_once(g, m, r, k, 5, 6, offset=chunks % 4)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, 5, 6), f"chunks={chunks} {ops}")
    if ops == "rtopk":
        # with k = r everything is sent and nothing left out, from the same sample
        every = u.gpu_encode_once(g, m, r, r, 5, 6, offset=chunks % 4)[3]["superset_size"]
        assert got[3]["path"] == 0 and (got[3]["superset_size"] == every) == whole, (got[3], every)


@pytest.mark.parametrize("d,r,whole", [(1 << 21, (1 << 17) - 1, True), (1 << 21, 1 << 17, False),
                                       (1 << 20, 1 << 17, True), ((1 << 20) + 1, 1 << 17, False),
                                       (4096 * 1024, 1 << 17, False)])
def test_short_vectors_with_many_candidates_are_keyed(d, r, whole):
    """From 2^17 members per launch on a short vector's stream keys its candidates, unless
    they are an eighth of the vector; two vectors with half of them each do so together."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    rng = np.random.default_rng(d + r)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    g[::50] *= np.float32(1e4)                       # far above the rest
    m = np.zeros(d, np.float32)
    k = r // 10
    got = u.gpu_encode_once(g, m, r, k, 5, 6)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, 5, 6), f"d={d} r={r}")
    every = u.gpu_encode_once(g, m, r, r, 5, 6)[3]["superset_size"]
    assert got[3]["path"] == 0 and (got[3]["superset_size"] == every) == whole, (got[3], every)
    r, k = (r + 1) // 2, r // 20
    grads = [torch.from_numpy(g).to(u.DEV) for _ in range(2)]
    res = [torch.zeros(d, device=u.DEV) for _ in range(2)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(2)]
    val = [torch.empty(k, device=u.DEV) for _ in range(2)]
    ws = torch.empty(2 * rt.encode_workspace_bytes(d, r, k), dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.encode_batch(grads, res, r, k, [5, 8], 6, idx, val, ws)
    torch.cuda.synchronize()
    for w, seed in enumerate((5, 8)):
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, m, r, k, seed, 6), f"batch of two, d={d} member {w}")


@pytest.mark.parametrize("n", [15, 16])
def test_short_random_k_batches_on_both_sides_of_keying(n):
    """r == d: from 2^23 elements per launch on a short vector's stream leaves the keys it
    computes anyway in the candidate buffer."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    d, k = 1 << 19, 5000
    rng = np.random.default_rng(n)
    g = rng.standard_normal(d).astype(np.float32)
    m = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    grad = torch.from_numpy(g).to(u.DEV)
    res = [torch.from_numpy(m).to(u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, d, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.encode_batch([grad] * n, res, d, k, list(range(n)), 6, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        assert rt.encode_stats(ws[w * stride:(w + 1) * stride])["path"] == 0
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, m, d, k, w, 6), f"member {w} of {n}")


@pytest.mark.parametrize("n,d,r", [(4, 2303 * 1024, 9000), (4, 2303 * 1024 + 1, 9000), (3, 3072 * 1024, 9000),
                                   (3, 3071 * 1024, 9000), (4, 3327 * 1024, 20000), (4, 3327 * 1024 + 1, 20000),
                                   (4, 4500 * 1024, 4500 * 32), (4, 4500 * 1024, 4500 * 32 + 1), (6, 4500 * 1024, 9000)])
def test_batches_around_the_changes_of_shape_and_share_out(n, d, r):
    """Chunks in all, and chunks, candidates and members per launch, on both sides of
    where the streaming kernel changes its shape and the walking kernels their share-out."""
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    k = r // 7
    rng = np.random.default_rng(d + n)
    gs = [(rng.standard_normal(d) * 10.0 ** rng.uniform(-3, 0, d)).astype(np.float32) for _ in range(2)]
    m = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    dev = [torch.from_numpy(g).to(u.DEV) for g in gs]
    res = [torch.from_numpy(m).to(u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.encode_batch([dev[w % 2] for w in range(n)], res, r, k, list(range(n)), 3, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        st = rt.encode_stats(ws[w * stride:(w + 1) * stride])
        assert st["path"] == 0 and st["error_flags"] == 0, (w, st)
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        if w in (0, n - 1):
            u.assert_encode_equal(got, oracle.encode(gs[w % 2], m, r, k, w, 3), f"member {w} of {n}, d={d} r={r}")


@pytest.mark.parametrize("d", [2_000_003, 3_000_001, 4_000_000])
def test_short_vectors_sample_enough_for_a_heavy_tail(d):
    """Below 2^22 elements the estimate takes as many samples as put 160 into the top r: its
    bracket then ends at a sample of rank 50 or so and not at the largest one or two, which
    in a heavy-tailed vector lie far above. About 1.4 r entries lie in the bracket, over 256
    linear bins of which rounding to a power of two leaves half: 3 r / 256 in the deciding
    bin, and not twice that (80 samples: 7 r / 256)."""
    from tests import gpu_util as u
    rng = np.random.default_rng(d)
    g = rng.standard_t(3, d).astype(np.float32)
    m = np.zeros(d, np.float32)
    r, k = d // 100, d // 1000
    got = u.gpu_encode_once(g, m, r, k, 42, 1)
    u.assert_encode_equal(got, oracle.encode(g, m, r, k, 42, 1), f"d={d}")
    assert got[3]["path"] == 0 and got[3]["boundary_list_size"] <= 5 * r // 256, got[3]


@pytest.mark.parametrize("d", [1, 1023, 1024, 1025, 100_003, 2049 * 1024, 2050 * 1024 - 1, 3500 * 1024 + 511,
                               4097 * 1024 + 1, (1 << 25) + 1700])
def test_the_calibration_add_covers_every_element_once(d):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    gen = torch.Generator(device=u.DEV).manual_seed(d)
    g, m = (torch.randn(d + 64, generator=gen, device=u.DEV) for _ in range(2))
    want = m.clone()
    want[:d] += g[:d]
    rt.diag_stream_add(g[:d], m[:d])
    assert torch.equal(m, want)
