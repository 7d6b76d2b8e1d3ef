"""Windows inside and across 64-sample blocks where most samples are above the
threshold: triggers identical to the oracle's on both sides of the one-launch limit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [64, 129, 4000, 8192, 20001])
@pytest.mark.parametrize("W", [1, 2, 15, 31, 32, 33, 61, 62])
def test_dense_triggers(n, W):
    from paper_1602_05573_amd import cluster_triggers
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    rng = np.random.default_rng(n + W)
    for levels in (3, 40, 100000):   # plateaus, ties, few ties
        M = rng.integers(0, levels + 1, n).astype(np.float32) / np.float32(levels)
        M[rng.integers(0, n, 3)] = (np.nan, np.inf, -np.inf)
        J = rng.integers(0, 1000, n).astype(np.int32)
        print("[case] dense n=%d W=%d levels=%d" % (n, W, levels), flush=True)
        md, jd = torch.from_numpy(M).cuda(), torch.from_numpy(J).cuda()
        for thr in (0.0, 0.4):
            ri, rt, rv = oracle.clusters(M, J, thr, W)
            i, t, v, total = cluster_triggers(md, jd, thr, W)
            assert total == len(ri)
            assert np.array_equal(i.cpu().numpy(), ri) and np.array_equal(t.cpu().numpy(), rt)
            assert np.array_equal(v.cpu().numpy().view(np.uint32), rv.view(np.uint32))
