"""One vector of medium length is sampled by need: lengths, top sets and batch sizes on both sides of where
that begins. The bracket holds the threshold (the ordinary path) and the message is the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,share", [(1, (1 << 22) - 1, 100), (1, 1 << 22, 100), (1, (1 << 22) + 3, 32), (1, (1 << 22) + 3, 31),
                                       (1, 6_000_001, 4000), (1, 1 << 24, 100), (1, (1 << 24) + 1, 100), (2, 5_000_001, 100)])
@pytest.mark.parametrize("values", ["layers", "student"])
def test_sample_by_need(n, d, share, values):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    rng = np.random.default_rng(d + share)
    if values == "student":
        g = rng.standard_t(3, d).astype(np.float32)
    else:
        g = (rng.standard_normal(d) * np.repeat(10.0 ** rng.uniform(-4, -1, 64), -(-d // 64))[:d]).astype(np.float32)
    r = d // share
    k = r // 5
    print(f"samples n={n} d={d} r={r} {values}", flush=True)
    grad = torch.from_numpy(g).to(u.DEV)
    res = [torch.zeros(d, device=u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.encode_batch([grad] * n, res, r, k, list(range(4, 4 + n)), 6, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        st = rt.encode_stats(ws[w * stride:(w + 1) * stride])
        assert st["path"] == 0 and st["error_flags"] == 0, st
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, np.zeros(d, np.float32), r, k, 4 + w, 6), f"member {w} of {n}")


@pytest.mark.parametrize("d,sampled", [(1 << 20, False), ((1 << 20) + 1, True), ((1 << 20) + 1023, True)])
@pytest.mark.parametrize("r", [40, 20_000, 200_000])
def test_the_shortest_strata(d, sampled, r):
    """Vectors of up to 1024 chunks have no sample; the shortest that may (they are counted otherwise) have strata of 64
    elements: 16,384 locations where r is small, fewer for larger r."""
    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    rng = np.random.default_rng(d + r)
    g = rng.standard_normal(d).astype(np.float32)
    m = (rng.standard_normal(d) * 1e-2).astype(np.float32)
    w = u.GpuWorker(d, r, r // 4, residual=m, offset=d % 4)
    got = w.encode(g, 3, 9, force=rt.FORCE_BRACKET_LOW)
    u.assert_encode_equal(got, oracle.encode(g, m, r, r // 4, 3, 9), f"d={d} r={r}")
    assert (u.estimated_bins(w.ws) != 0) == sampled
