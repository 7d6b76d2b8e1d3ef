"""Multi-rate bank at the edges of its launches: interpolation tap counts around
the two-tap-pair step, rows of odd stride, levels of one segment grouped with
levels of many (state passes composed inline and by the chain launch), and a
large level beside the group; against the oracle's definition."""
import numpy as np
import pytest

import oracle
from helpers import SNR_TOL
from test_gpu_multirate import rand_levels, z_err
from workloads import strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


def run(levels, lh, lg, x, cuts, max_block, seed, trigger=False):
    from paper_1602_05573_amd import SpiirMultiRate
    rng = np.random.default_rng(seed)
    h, g = rng.standard_normal(lh) / lh, rng.standard_normal(lg) / lg
    ref = oracle.multirate_z(levels, h, g, x)
    xd = torch.from_numpy(x).cuda()
    with SpiirMultiRate(levels, h, g, max_block=max_block) as mr:
        z = torch.cat([mr.filter_block_z(xd[a:b].contiguous()) for a, b in zip(cuts[:-1], cuts[1:])], dim=1)
        err = z_err(z.cpu().numpy(), ref)
        mr.reset()
        mx = torch.cat([mr.trigger_max(xd[a:b].contiguous())[0] for a, b in zip(cuts[:-1], cuts[1:])])
    s = (ref.real ** 2 + ref.imag ** 2).max(axis=0)
    print("z error %.3g" % err, flush=True)
    assert err <= SNR_TOL
    assert np.max(np.abs(mx.cpu().numpy() - s)) <= SNR_TOL * s.max()


@pytest.mark.parametrize("lg", [1, 2, 3, 4, 5, 6, 7, 63, 64])
def test_interpolation_taps(lg):
    print("[case] interpolation taps %d" % lg, flush=True)
    x = strain(4096, 7, lg)
    run(rand_levels(18, [5, 0, 7, 9], lg), 24, lg, x, [0, 512, 520, 2568, 4096], 2048, lg)


def test_odd_rows():
    print("[case] odd rows", flush=True)
    run(rand_levels(5, [20], 1), 8, 8, strain(3003, 7, 1), [0, 1, 1002, 3003], 1001, 1)


@pytest.mark.parametrize("n,mb", [(64, 64), (512, 512), (8192, 8192), (16384, 16384)])
def test_group_of_levels(n, mb):
    """Levels of 1 segment (n >> 4 samples) to more than 16 (n samples) in one group."""
    print("[case] group n=%d" % n, flush=True)
    x = strain(3 * n, 7, n)
    run(rand_levels(7, [30, 12, 0, 9, 25], n), 24, 24, x, [0, n, 2 * n, 2 * n + n // 2, 3 * n], mb, n)


def test_large_level_beside_the_group():
    print("[case] large level", flush=True)
    x = strain(3000, 7, 3)
    run(rand_levels(260, [40, 260, 30], 3), 24, 24, x, [0, 2048, 2052, 3000], 2048, 3)


@pytest.mark.parametrize("lh,levels,n,mb", [(1, 4, 2048, 1024), (2, 3, 3000, 2000), (24, 8, 8192, 4096),
                                            (64, 8, 4096, 2048), (7, 2, 1030, 1030)])
def test_decimation_slices(lh, levels, n, mb):
    """Slices of 512 samples: one, several, a short last one; reaches from none to many slices."""
    print("[case] decimation taps %d levels %d" % (lh, levels), flush=True)
    per = [0] * (levels - 1) + [12]
    step = 1 << (levels - 1)
    x = strain(n, 7, lh)
    run(rand_levels(4, per, lh), lh, 8, x, [0, step, mb // (2 * step) * step + step, n], mb, lh)
