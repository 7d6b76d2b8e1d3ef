"""Full passes in batches of 64, 32, 16 and 8 steps (as many as the row sums find LDS
for beside the delays), chunk lengths that 16 does not divide, and a bank whose window
goes to global memory because it would take another round of workgroups in LDS: rows,
keys, the allocation-free call, the comparator and batches against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from helpers import SNR_TOL, check_argmax, snr_err
from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


# delays whose window leaves LDS for 64, 32, 16, 8 steps of 8 waves
@pytest.mark.parametrize("dmax", [20000, 25000, 29500, 31000])
@pytest.mark.parametrize("L", [256, 24])
def test_batch_lengths(dmax, L):
    from paper_1602_05573_amd import SpiirBank
    bank = random_bank(105, dmax + L, 6, 30, 200 if dmax < 31000 else 300, 0.99, 1 - 1e-5, dmax)
    cuts = np.cumsum([0, 1, 15, 66, 200, 517, 2048])
    x = strain(int(cuts[-1]), 105, dmax)
    ref = oracle.snr(bank, x)
    xd = torch.from_numpy(x).cuda()
    parts = [xd[a:b].contiguous() for a, b in zip(cuts[:-1], cuts[1:])]
    for ts in (1, 3):
        print("[case] batches, delays %d L %d time_split %d" % (dmax, L, ts), flush=True)
        with SpiirBank.from_bank(bank, chunk_len=L, filters_per_lane=1 if dmax < 31000 else 3,
                                 waves_per_group=8, time_split=ts) as bk:
            assert bk.info["x_in_lds"] == 1
            rows = torch.cat([bk.filter_block(p) for p in parts], dim=1)
            assert snr_err(rows.cpu().numpy(), ref)[0] <= SNR_TOL
            for call in (bk.trigger_max, bk.trigger_max_per_template):
                bk.reset()
                out = [call(p) for p in parts]
                check_argmax(*(torch.cat([o[i] for o in out]).cpu().numpy() for i in (0, 1)), ref)


def test_window_that_would_take_another_round():
    """260 workgroups of 8 waves on 256 compute units."""
    from paper_1602_05573_amd import SpiirBank, SpiirBatch
    bank = random_bank(106, 0, 520, 250, 250, 0.99, 1 - 1e-5, 25000)
    n = 3000
    x = strain(n, 106)
    ref = oracle.snr(bank, x, nthreads=oracle.max_threads())
    xd = torch.from_numpy(x).cuda()
    opts = dict(filters_per_lane=1, waves_per_group=8, max_block=8192)
    print("[case] window in global memory to save a round", flush=True)
    with SpiirBank.from_bank(bank, **opts) as bk:
        if bk.info["n_cu"] == 256:
            assert bk.info["n_groups"] == 260 and bk.info["x_in_lds"] == 0
        rows = torch.cat([bk.filter_block(xd[:1000].contiguous()), bk.filter_block(xd[1000:].contiguous())], dim=1)
        assert snr_err(rows.cpu().numpy(), ref)[0] <= SNR_TOL
        # calls whose window does not fit the allocation-free array run with it in LDS
        bk.reset()
        many = (32 << 20) // 4
        big = torch.zeros(many, device="cuda")
        big[:n] = xd
        m, j = torch.empty(many, device="cuda"), torch.empty(many, dtype=torch.int32, device="cuda")
        bk.trigger_max_noalloc(big, out=(m, j))
        check_argmax(m[:n].cpu().numpy(), j[:n].cpu().numpy(), ref)
    # a first call under capture has no window to allocate, nor has a forward without a tape
    with SpiirBank.from_bank(bank, **opts) as bk:
        snr = torch.empty((bank.n_templates, n), device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            bk.filter_block(xd, snr, stream=side)
            z = bk.forward_z(xd, stream=side)
        graph.replay()
        torch.cuda.synchronize()
        assert snr_err(snr.cpu().numpy(), ref)[0] <= SNR_TOL
        z = (z[0] if isinstance(z, tuple) else z).cpu().numpy()
        assert snr_err(z.real ** 2 + z.imag ** 2, ref)[0] <= SNR_TOL
        del graph
    # a batch stages the window in LDS all the same
    banks = [SpiirBank.from_bank(bank, **opts) for _ in range(2)]
    bt = SpiirBatch(banks, [xd, xd[:1500].contiguous()], block_len=1024)
    for _ in range(bt.steps_total()):
        bt.step()
    torch.cuda.synchronize()
    check_argmax(bt.max[0].cpu().numpy(), bt.argmax[0].cpu().numpy(), ref)
    assert float((bt.max[1] - bt.max[0][:1500]).abs().max()) <= SNR_TOL * float(bt.max[0].max())
    bt.close()
    for bk in banks:
        bk.close()
