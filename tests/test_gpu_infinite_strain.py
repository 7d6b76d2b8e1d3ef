"""An infinite sample: every output before it reaches a template's first filter is what
it is without it, the output at that sample is infinite, later ones are NaN (the
state is), at every position inside a block of steps, with the window in LDS and
in global memory, whole and cut into segments, in a call and in the history of the next."""
import numpy as np
import pytest

import oracle
from helpers import SNR_TOL
from workloads import Bank, random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("fl", [1, 2, 3, 4])
@pytest.mark.parametrize("dmax,ts", [(400, 1), (400, 0), (400, 3), (60000, 1), (60000, 0)])
def test_first_output_is_infinite(fl, dmax, ts):
    from paper_1602_05573_amd import SpiirBank
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    K, T, n, cut = 16 * fl, 5, 3000, 1200   # whole rows: no padding slots
    bank = random_bank(110, fl, T, K, K, 0.95, 0.999, 400)
    d = bank.d.copy()
    first = np.array([3, 10, 17, 24, 150])   # every position of a 4-step block and a later one
    for j in range(T):
        sl = slice(int(bank.offsets[j]), int(bank.offsets[j + 1]))
        d[sl] = np.maximum(d[sl], first[j] + 1)
        d[sl.start] = first[j]
    bank = Bank(bank.offsets, bank.a, bank.b, d, dmax)
    x = strain(n, 110, fl)
    ref = oracle.snr(bank, x)
    print("[case] infinite sample, fl %d delays %d time_split %d" % (fl, dmax, ts), flush=True)
    with SpiirBank.from_bank(bank, filters_per_lane=fl, time_split=ts) as bk:
        for at, v in ((700, np.inf), (701, -np.inf), (1100, np.inf), (1199, np.inf), (1200, np.inf)):
            y = x.copy()
            y[at] = v
            xd = torch.from_numpy(y).cuda()
            bk.reset()
            s = torch.cat([bk.filter_block(xd[:cut].contiguous()), bk.filter_block(xd[cut:].contiguous())], dim=1)
            s = s.cpu().numpy()
            for j in range(T):
                t = at + int(first[j])
                assert np.abs(s[j, :t] - ref[j, :t]).max() <= SNR_TOL * ref[j].max()
                assert np.isposinf(s[j, t]), "template %d sample %d" % (j, t)
                assert np.isnan(s[j, t + 1:]).all()
            bk.reset()
            m, _ = bk.trigger_max(xd[:cut].contiguous())
            m2, _ = bk.trigger_max(xd[cut:].contiguous())
            m = torch.cat([m, m2]).cpu().numpy()
            assert np.isfinite(m[:at + 3]).all() and np.isposinf(m[at + 3]) and np.isnan(m[at + 4:]).all()
            if dmax == 400:
                z, tape = bk.forward_z(xd, want_tape=True)
                tape.close()
                z = z.cpu().numpy()
                assert all(np.isinf(z[j, at + first[j]].real) and np.isinf(z[j, at + first[j]].imag) for j in range(T))
