"""How the streaming kernel's chunks are dealt to its wavefronts, on both sides of
where that changes. Against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,top", [(2, (1 << 23) - 1, 1.0), (2, 1 << 23, 1.0), (1, (1 << 23) + 1700, 1.0),
                                     (1, 4100 * 1024 + 3, 0.01), (2, 4100 * 1024 + 3, 0.01),
                                     (1, 1 << 26, 0.001), (1, (1 << 26) + 1, 0.001)])
def test_every_chunk_is_dealt_once(n, d, top):
    import torch

    import paper_2005_10761_amd as rt
    from tests import gpu_util as u
    r = int(d * top)
    k = r // 50
    rng = np.random.default_rng(d + n)
    g = rng.standard_normal(d, dtype=np.float32)
    m = rng.standard_normal(d, dtype=np.float32) * np.float32(1e-3)
    print(f"dealing n={n} d={d} r={r}", flush=True)
    grad = torch.from_numpy(g).to(u.DEV)
    res = [torch.from_numpy(m).to(u.DEV) for _ in range(n)]
    idx = [torch.empty(k, dtype=torch.int32, device=u.DEV) for _ in range(n)]
    val = [torch.empty(k, device=u.DEV) for _ in range(n)]
    stride = rt.encode_workspace_bytes(d, r, k)
    ws = torch.empty(n * stride, dtype=torch.uint8, device=u.DEV).fill_(0xA5)
    rt.encode_batch([grad] * n, res, r, k, list(range(7, 7 + n)), 6, idx, val, ws)
    torch.cuda.synchronize()
    for w in range(n):
        assert rt.encode_stats(ws[w * stride:(w + 1) * stride])["path"] == 0
        got = (idx[w].cpu().numpy().view(np.uint32), val[w].cpu().numpy(), res[w].cpu().numpy())
        u.assert_encode_equal(got, oracle.encode(g, m, r, k, 7 + w, 6), f"member {w} of {n}, d={d} r={r}")
