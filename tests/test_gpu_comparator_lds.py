"""The per-template comparator on banks whose plan for short segments sums in
larger batches than their plan for whole pieces (chunk lengths that do not
divide 2,048, delays near the LDS limit), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from helpers import check_argmax
from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,dmax,opts", [(384, 36278, {}), (1536, 34000, dict(waves_per_group=2)),
                                         (768, 22000, dict(waves_per_group=8))])
def test_comparator_near_the_lds_limit(L, dmax, opts):
    from paper_1602_05573_amd import SpiirBank
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    bank = random_bank(101, L, 5, 20, 60, 0.99, 1 - 1e-5, dmax)
    n = 3 * L + 137
    cuts = [0, L + 65, n, dmax + n]
    x = strain(cuts[-1], 101, L)
    ref = oracle.snr(bank, x)
    print("[case] comparator L %d delays %d %s" % (L, dmax, opts), flush=True)
    xd = torch.from_numpy(x).cuda()
    with SpiirBank.from_bank(bank, chunk_len=L, **opts) as bk:
        outs = [bk.trigger_max_per_template(xd[a:b].contiguous()) for a, b in zip(cuts[:-1], cuts[1:])]
    mx, am = (torch.cat([o[i] for o in outs]).cpu().numpy() for i in (0, 1))
    check_argmax(mx, am, ref)
