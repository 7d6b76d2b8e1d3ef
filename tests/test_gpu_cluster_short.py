"""Clustering of short series in one workgroup, and of the longest and shortest
series on both sides of that: identical to the oracle's plain window scan."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


def series(n, seed, levels):
    """Values on few levels, so that ties and plateaus are common."""
    rng = np.random.default_rng(seed)
    M = rng.integers(-levels, levels + 1, n).astype(np.float32) / np.float32(levels)
    if n > 40:
        M[n // 3] = np.nan
        M[n // 2] = np.inf
        M[n // 2 + n // 5] = -np.inf
        M[5:12] = 3.0
    return M, rng.integers(0, 1000, n).astype(np.int32)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("W", [0, 1, 2, 7, 33, 62, 63, 64, 129, 5000, 2**31 - 1])
def test_short_series(n, W):
    from paper_1602_05573_amd import cluster_triggers
    for levels in (2, 100000):
        M, J = series(n, n + W, levels)
        print("[case] short n=%d W=%d levels=%d" % (n, W, levels), flush=True)
        md, jd = torch.from_numpy(M).cuda(), torch.from_numpy(J).cuda()
        for thr in (-np.inf, -0.5, 0.0, 0.9):
            ri, rt, rv = oracle.clusters(M, J, float(thr), W)
            for cap in (None, len(ri) // 2):
                i, t, v, total = cluster_triggers(md, jd, float(thr), W, capacity=cap)
                assert total == len(ri)
                k = len(i)
                assert np.array_equal(i.cpu().numpy(), ri[:k])
                assert np.array_equal(t.cpu().numpy(), rt[:k])
                assert np.array_equal(v.cpu().numpy().view(np.uint32), rv[:k].view(np.uint32))
        assert cluster_triggers(md, jd, float("nan"), W)[3] == 0


@pytest.mark.parametrize("W,blocks", [(0, [1, 5000, 300]), (100, [8092, 1, 7900, 5000, 8000, 70]),
                                      (3000, [2192, 2193, 5000, 100, 2192, 2193, 7000])])
def test_stream_around_the_short_limit(W, blocks):
    """Pushes whose joined window is on both sides of the limit of a short series."""
    from paper_1602_05573_amd import TriggerStream
    n = sum(blocks)
    M, J = series(n, W + 1, 100000)
    M[np.isnan(M)] = 0.0
    ri, rt, rv = oracle.clusters(M, J, 0.2, W)
    print("[case] stream W=%d" % W, flush=True)
    got, p = [], 0
    ts = TriggerStream(0.2, W, max(blocks), capacity=n + 1)
    for b in blocks:
        got.append(ts.push(torch.from_numpy(M[p:p + b].copy()).cuda(), torch.from_numpy(J[p:p + b].copy()).cuda()))
        p += b
    got.append(ts.flush())
    ts.close()
    i, t, v = (torch.cat([g[q] for g in got]).cpu().numpy() for q in range(3))
    assert np.array_equal(i, ri) and np.array_equal(t, rt)
    assert np.array_equal(v.view(np.uint32), rv.view(np.uint32))
