"""Batches of banks whose plans sum in batches of different length (a bank cut into
short segments beside one that is not, delays near the LDS limit) run and match
the FP64 oracle; chunk lengths of both classes are still refused."""
import pytest

import oracle
from helpers import check_argmax
from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_plans_of_different_batch_length():
    from paper_1602_05573_amd import SpiirBank, SpiirBatch, SpiirError
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    opts = dict(filters_per_lane=1, waves_per_group=1)
    specs = [(384, 36278, dict(time_split=0)), (384, 36278, dict(time_split=1)), (256, 36900, dict(time_split=1))]
    lengths = (40000, 39001, 38400)
    banks = [random_bank(107, i, 3, 20, 60, 0.99, 1 - 1e-5, d) for i, (_, d, _) in enumerate(specs)]
    xs = [strain(n, 107, i) for i, n in enumerate(lengths)]
    bks = [SpiirBank.from_bank(b, chunk_len=L, **opts, **o) for b, (L, _, o) in zip(banks, specs)]
    print("[case] batch of plans with different batch lengths", flush=True)
    for mode in (1, 2):
        bt = SpiirBatch(bks, [torch.from_numpy(x).cuda() for x in xs], block_len=1024)
        bt.set_time_split(mode)
        for _ in range(bt.steps_total()):
            bt.step()
        torch.cuda.synchronize()
        for b, x, m, j in zip(banks, xs, bt.max, bt.argmax):
            check_argmax(m.cpu().numpy(), j.cpu().numpy(), oracle.snr(b, x))
        bt.reset()
        torch.cuda.synchronize()
        bt.close()
    short = SpiirBank.from_bank(banks[0], chunk_len=24, **opts)
    with pytest.raises(SpiirError, match="tile length"):
        SpiirBatch([bks[0], short], [torch.from_numpy(x).cuda() for x in xs[:2]], block_len=1024)
    for bk in bks + [short]:
        bk.close()
