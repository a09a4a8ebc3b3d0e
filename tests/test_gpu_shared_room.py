"""Where the rules around the candidate buffer, the short lists and the dense
average's runs of tiles change over. Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _encode(g, r, k, seed, steps=2, offset=0):
    from tests import gpu_util as u
    d = len(g)
    w, res, paths = u.GpuWorker(d, r, k, offset=offset), np.zeros(d, np.float32), []
    for t in range(steps):
        got = w.encode(g, seed, t)
        oi, ov, res = oracle.encode(g, res, r, k, seed, t)
        u.assert_encode_equal(got, (oi, ov, res), f"d={d} r={r} k={k} step {t}")
        paths.append(w.stats["path"])
    return paths


def _stride(d):
    """Elements between two chunks of one streaming wavefront: 2048 wavefronts up to 4096 chunks, 3072 above."""
    return (2048 if d <= 4096 * 1024 else 3072) * 1024


@pytest.mark.parametrize("d", [3_200_700, 6_300_001, 9_500_123])      # 1 to 2 chunks per wavefront of 2048; 2 to 3, 3 to 4 of 3072
@pytest.mark.parametrize("hot", ["first", "last", "ragged", "same_wavefront", "all_of_one"])
@pytest.mark.parametrize("k_of_r", [1, 2, 5])
def test_chunks_share_their_wavefronts_room(d, hot, k_of_r):
    """Chunks that are members throughout, at the ends of a wavefront's part of the buffer, two of one
    wavefront, and all of one wavefront's. Up to 4096 chunks the stream keeps all of such a chunk, which never
    fits; above, it keeps what may be sent: all with k = r, a half or a quarter else."""
    stride = _stride(d)
    rng = np.random.default_rng(d + k_of_r)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    starts = {"first": [0], "last": [(d // 1024 - 1) * 1024], "ragged": [d // 1024 * 1024],
              "same_wavefront": [5 * 1024, 5 * 1024 + stride], "all_of_one": range(7 * 1024, d, stride)}[hot]
    hot_chunks = 0
    for s in starts:
        n = len(g[s:s + 1024])
        assert n > 300                                                # (a hot chunk, also at the ragged end)
        g[s:s + 1024] = rng.standard_normal(n).astype(np.float32) * 5.0 + np.float32(20.0)
        hot_chunks += 1
    assert hot_chunks == {"all_of_one": -(-(d - 7 * 1024) // stride), "same_wavefront": 2}.get(hot, 1)
    r = 5_000
    print(f"shared room d={d} hot={hot} r={r} k={r // k_of_r}", flush=True)
    _encode(g, r, r // k_of_r, 3, offset=d % 4)


@pytest.mark.parametrize("d", [3_200_700, 6_300_001])                 # candidates without their keys, and with them
@pytest.mark.parametrize("count", [127, 128, 129, 191, 192, 193, 300])
def test_room_left_by_the_wavefronts_other_chunk(d, count):
    """A wavefront's two chunks have room for 2 * 128 entries, of which the first may take 192. The entries of
    both are looked for in the workspace: what fits is there whole (so a share beyond 128 was taken), and of a
    first chunk that does not fit, what the second one's slice, which then starts at the same place, left over."""
    from tests import gpu_util as u
    torch = u.torch
    r, k, seed, second_count = 5_000, 2_500, 3, 60
    rng = np.random.default_rng(d + count)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    patterns = []
    for chunk, n in ((100, count), (100 + _stride(d) // 1024, second_count)):
        c0 = chunk * 1024
        # certain winners, which every stream keeps: the window lies around half of the keys
        sure = [i for i in range(c0, c0 + 1024) if oracle.key64(seed, 0, i) < int(0.4 * 2**64)]
        places = np.sort(rng.permutation(np.array(sure))[:n])
        assert len(places) == n
        g[c0:c0 + 1024] = 0.0
        # (low bits set: two samples of the estimate, the upper halves of two patterns, make no such word)
        g[places] = (20.0 + 3 / 2**18 + chunk / 64 + np.arange(n) / 1024).astype(np.float32)
        assert np.all(g[places].view(np.uint32) & 0xFF != 0)
        patterns.append(torch.from_numpy(g[places].view(np.int32)).to(u.DEV))
    print(f"room left d={d} count={count}", flush=True)
    w = u.GpuWorker(d, r, k)
    got = w.encode(g, seed, 0)
    u.assert_encode_equal(got, oracle.encode(g, np.zeros(d, np.float32), r, k, seed, 0), f"d={d} count={count}")
    words = w.ws.view(torch.int32)
    first, second = (int(torch.isin(p, words).sum()) for p in patterns)
    assert second == second_count
    assert first == (count if count <= 192 else 192 - second_count), (first, count)


@pytest.mark.parametrize("d,r,k,levels", [(200_003, 4_000, 900, 64), (200_003, 12_000, 1_500, 8), (1_048_576, 10_485, 1_048, 4),
                                          (1_500_000, 1_500, 1_500, 4), (70_001, 300, 60, 1024), (4_200_000, 40_000, 8_000, 16)])
def test_deciding_bin_of_a_few_levels(d, r, k, levels):
    """Quantised values: from a handful to thousands of equal magnitudes share the bin of the cut, in lists
    that fit the staging area and lists that do not."""
    g = (np.round(np.random.default_rng(d + r).standard_normal(d) * levels) / levels).astype(np.float32)
    print(f"levels d={d} r={r} k={k} levels={levels}", flush=True)
    assert not any(p & 2 for p in _encode(g, r, k, 11))


@pytest.mark.parametrize("d,hot,r,k", [(1 << 20, 4600, 4600, 2300), (1 << 20, 4600, 4590, 4000), (1 << 20, 4608, 4608, 2304),
                                       (1 << 20, 4609, 4609, 2304), (2_000_003, 4600, 4600, 2300), (1 << 20, 4600, 4600, 4600)])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_nearly_all_members_in_the_deciding_bin(d, hot, r, k, seed):
    """Entries of +-1 at random places over small noise: the top r lies in the deciding bin but for nothing, and
    some 540 of its keys join those in the window (k = r: none)."""
    rng = np.random.default_rng(d + hot + seed)
    g = (rng.standard_normal(d) * 1e-3).astype(np.float32)
    g[rng.permutation(d)[:hot]] = rng.choice(np.array([-1.0, 1.0], np.float32), hot)
    print(f"deciding bin d={d} hot={hot} r={r} k={k} seed={seed}", flush=True)
    assert not any(p & 3 for p in _encode(g, r, k, seed, steps=1))


@pytest.mark.parametrize("k", [2_500_000, 3_500_000])
def test_more_keys_than_the_staging_area_holds(k):
    """Random-k whose key window holds 21,500 keys, which nearly fill the staging area, and 25,100 (23,936 are staged)."""
    d = 40_000_003
    g = np.random.default_rng(4).standard_normal(d).astype(np.float32)
    print(f"key list d={d} k={k}", flush=True)
    assert _encode(g, d, k, 5, steps=1) == [0]


@pytest.mark.parametrize("r,k", [(1, 1), (2, 1), (300, 1), (300, 299), (300, 300), (3_000, 40), (60_000, 59_999), (60_000, 30_000),
                                 (300_007, 1), (300_007, 150_000), (300_007, 300_006)])
def test_room_for_the_window_as_sizes_go(r, k):
    """The room for keys follows the window's width: one-sided windows, all but one sent, half, none looked at."""
    g = np.random.default_rng(r + k).standard_normal(300_007).astype(np.float32)
    print(f"room r={r} k={k}", flush=True)
    assert not any(p & 2 for p in _encode(g, r, k, 9))


@pytest.mark.parametrize("tiles", [4096, 4097, 12289, 28672, 28673])  # runs of one, two, four and seven tiles; of eight,
@pytest.mark.parametrize("per_tile", [1, 64])                         # which up to four workers cut to four
@pytest.mark.parametrize("n", [1, 4, 5])
def test_dense_average_over_the_runs_of_tiles(tiles, per_tile, n):
    from tests import gpu_util as u
    d = (tiles - 1) * 2048 + 7
    k = tiles * per_tile // n + 1
    rng = np.random.default_rng(tiles + per_tile + n)
    idx = np.stack([np.unique(rng.integers(0, d, 2 * k))[:k] for _ in range(n)]).astype(np.uint32)
    idx[:, -1] = d - 1
    val = rng.standard_normal((n, k)).astype(np.float32)
    print(f"average tiles={tiles} per tile {per_tile} n={n}", flush=True)
    out = u.gpu_aggregate(idx, val, n, d)
    assert np.array_equal(u.bits(out), u.bits(oracle.aggregate_f32(idx, val, n, d)))


@pytest.mark.parametrize("tiles", [8192, 8193, 16384, 16385, 16386])  # runs of one, two and four tiles, whole and not
@pytest.mark.parametrize("n", [16, 17, 33, 64, 65])
def test_momentum_step_over_the_runs_of_tiles(tiles, n):
    from tests import gpu_util as u
    d = (tiles - 1) * 2048 + 7
    k = 2 * tiles // n + 1
    rng = np.random.default_rng(tiles + n)
    idx = np.stack([np.unique(rng.integers(0, d, 2 * k))[:k] for _ in range(n)]).astype(np.uint32)
    idx[:, -1] = d - 1
    val = rng.standard_normal((n, k)).astype(np.float32)
    omega = rng.standard_normal(d, dtype=np.float32)
    vel = rng.standard_normal(d, dtype=np.float32) * np.float32(0.01)
    print(f"momentum tiles={tiles} n={n}", flush=True)
    gw, gv = u.gpu_aggregate_update_momentum(idx, val, n, d, 0.1, 1.0, 0.9, omega, vel)
    ww, wv = oracle.aggregate_update_momentum_f32(idx, val, n, d, 0.1, 1.0, 0.9, omega, vel)
    assert np.array_equal(u.bits(gv), u.bits(wv)) and np.array_equal(u.bits(gw), u.bits(ww))
