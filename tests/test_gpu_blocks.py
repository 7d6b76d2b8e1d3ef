"""Edges of the forward kernels' blocks against the FP64 oracle: calls that end
inside a 4-step block, an 8-step tile, a 64-step batch; waves that run the
plain recursion (small |a|); time splits on both sides of the segment count
up to which the full pass composes its own start states; segments shorter than
a chunk. The gate is the repository's peak-normalised SNR tolerance for FP32
paths."""
import numpy as np
import pytest

import oracle
from helpers import SNR_TOL, check_argmax, snr_err
from workloads import Bank, random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


def run_rows(bank, x, cuts, **opts):
    from paper_1602_05573_amd import SpiirBank
    xd = torch.from_numpy(x).cuda()
    with SpiirBank.from_bank(bank, **opts) as bk:
        rows = [bk.filter_block(xd[a:b].contiguous()).cpu().numpy() for a, b in zip(cuts[:-1], cuts[1:])]
        bk.reset()
        outs = [bk.trigger_max(xd[a:b].contiguous()) for a, b in zip(cuts[:-1], cuts[1:])]
        info = bk.info
    mx = torch.cat([o[0] for o in outs]).cpu().numpy()
    am = torch.cat([o[1] for o in outs]).cpu().numpy()
    return np.concatenate(rows, axis=1), mx, am, info


def small_poles(bank, every):
    """The bank with every `every`-th pole replaced by one of modulus below 0.1, one of them 0."""
    a = bank.a.copy()
    k = np.arange(0, len(a), every)
    a[k] = 0.09 * np.exp(1j * np.linspace(0.1, 3.0, len(k)))
    a[0] = 0.0
    return Bank(bank.offsets, a, bank.b, bank.d, bank.dmax)


@pytest.mark.parametrize("fl", [1, 2, 3, 4])
@pytest.mark.parametrize("every", [0, 1, 97])
def test_ragged_calls(fl, every):
    bank = random_bank(91, fl, 7, 3, 200, 0.99, 1 - 1e-5, 333)
    if every:
        bank = small_poles(bank, every)
    cuts = np.cumsum([0, 1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 130, 253, 258])
    x = strain(int(cuts[-1]), 91, fl)
    ref = oracle.snr(bank, x)
    for ts, L in ((1, 256), (1, 8), (3, 64)):
        print("[case] fl %d every %d time_split %d L %d" % (fl, every, ts, L), flush=True)
        s, mx, am, _ = run_rows(bank, x, cuts, filters_per_lane=fl, time_split=ts, chunk_len=L)
        assert snr_err(s, ref)[0] <= SNR_TOL
        check_argmax(mx, am, ref)


@pytest.mark.parametrize("nseg", [2, 7, 8, 9, 17, 32])
def test_segment_counts(nseg):
    bank = random_bank(92, 0, 9, 40, 300, 0.99, 1 - 1e-6, 700)
    n = 64 * 40 + 5
    x = strain(2 * n, 92)
    ref = oracle.snr(bank, x)
    print("[case] %d segments" % nseg, flush=True)
    s, mx, am, info = run_rows(bank, x, [0, n, 2 * n], time_split=nseg, chunk_len=64, max_block=4096)
    assert info["time_split"] == nseg
    assert snr_err(s, ref)[0] <= SNR_TOL
    check_argmax(mx, am, ref)


@pytest.mark.parametrize("n", [65, 129, 500, 513, 577, 1000, 4097, 16384])
@pytest.mark.parametrize("every", [0, 50])
def test_automatic_segments(n, every):
    """A small bank, whose calls are cut into as many segments as pay (shorter
    than a chunk of 256 samples for short calls)."""
    bank = random_bank(93, 0, 3, 100, 130, 0.99, 1 - 1e-6, 2047)
    if every:
        bank = small_poles(bank, every)
    x = strain(3 * n, 93)
    ref = oracle.snr(bank, x)
    print("[case] calls of %d samples, small poles every %d" % (n, every), flush=True)
    s, mx, am, _ = run_rows(bank, x, [0, n, 2 * n, 3 * n])
    assert snr_err(s, ref)[0] <= SNR_TOL
    check_argmax(mx, am, ref)


@pytest.fixture(scope="module")
def long_delays():
    # above 128 filters per compute unit of a 256-unit device, delays of four bands
    bank = random_bank(94, 0, 84, 380, 420, 0.99, 1 - 1e-5, 60000)
    x = strain(5000, 94)
    return bank, x, oracle.snr(bank, x, nthreads=oracle.max_threads())


def test_automatic_delay_bands(long_delays):
    """A large bank whose delays do not fit LDS is cut by delay; streaming calls,
    the per-template comparator and the allocation-free call against the oracle."""
    from paper_1602_05573_amd import SpiirBank, SpiirBatch, SpiirError
    bank, x, ref = long_delays
    print("[case] automatic delay bands", flush=True)
    s, mx, am, info = run_rows(bank, x, [0, 1000, 1003, 5000])
    assert info["delay_band"] > 0 and info["x_in_lds"] == 1 and info["n_parts"] > 0
    assert snr_err(s, ref)[0] <= SNR_TOL
    check_argmax(mx, am, ref)
    xd = torch.from_numpy(x).cuda()
    with SpiirBank.from_bank(bank) as bk:
        outs = [bk.trigger_max_per_template(xd[a:b].contiguous()) for a, b in ((0, 700), (700, 5000))]
        check_argmax(torch.cat([o[0] for o in outs]).cpu().numpy(), torch.cat([o[1] for o in outs]).cpu().numpy(), ref)
        bk.reset()
        m = torch.empty(5000, dtype=torch.float32, device="cuda")
        j = torch.empty(5000, dtype=torch.int32, device="cuda")
        bk.trigger_max_noalloc(xd, out=(m, j))
        check_argmax(m.cpu().numpy(), j.cpu().numpy(), ref)
        with pytest.raises(SpiirError, match="outside LDS"):
            SpiirBatch([bk], [xd], block_len=4096)


@pytest.mark.parametrize("n,L,K", [(1, 256, 64), (15, 256, 65), (16, 8, 1), (17, 24, 63), (300, 256, 128), (1000, 64, 200)])
def test_backward_edges(n, L, K):
    """Gradients where sub-chunks, chunks and waves of the backward are partly
    filled; the gate is the one of the adjoint tests (per-template norm)."""
    from paper_1602_05573_amd import SpiirBank
    bank = random_bank(95, K, 5, K, K, 0.95, 0.9999, 90)
    x = strain(n, 95)
    zr = oracle.z(bank, x)
    rng = np.random.default_rng(95)
    G = (rng.standard_normal(zr.shape) + 1j * rng.standard_normal(zr.shape)).astype(np.complex64)
    ga_ref, gb_ref = oracle.backward(bank, x, G.astype(np.complex128))
    print("[case] backward n %d L %d K %d" % (n, L, K), flush=True)
    for ts in (1, 3):
        with SpiirBank.from_bank(bank, chunk_len=L, time_split=ts) as bk:
            z, tape = bk.forward_z(torch.from_numpy(x).cuda(), want_tape=True)
            ga, gb = bk.backward(tape, torch.from_numpy(G).cuda())
            tape.close()
            ga, gb = ga.cpu().numpy(), gb.cpu().numpy()
        for g, r in ((ga, ga_ref), (gb, gb_ref)):
            for j in range(bank.n_templates):
                sl = slice(int(bank.offsets[j]), int(bank.offsets[j + 1]))
                assert np.linalg.norm(g[sl] - r[sl]) <= 1e-3 * np.linalg.norm(r[sl])


def test_automatic_delay_bands_at_the_scratch_limit():
    """A banded bank whose keys for whole pieces exceed the allocation-free call's
    array runs that call in shorter pieces, with the same stream."""
    from paper_1602_05573_amd import SpiirBank
    bank = random_bank(96, 0, 1400, 400, 420, 0.99, 1 - 1e-5, 60000)
    x = torch.from_numpy(strain(16384, 96)).cuda()
    print("[case] automatic delay bands, scratch limit", flush=True)
    with SpiirBank.from_bank(bank) as bk:
        info = bk.info
        assert info["delay_band"] > 0 and info["n_groups"] * 16384 * 8 > 32 << 20
        mx, am = bk.trigger_max(x)
        bk.reset()
        m, j = torch.empty_like(mx), torch.empty_like(am)
        bk.trigger_max_noalloc(x, out=(m, j))
        tail = bk.trigger_max(x[:100].contiguous())[0]
        bk.reset()
        bk.trigger_max(x)
        want = bk.trigger_max(x[:100].contiguous())[0]
    assert float((m - mx).abs().max()) <= SNR_TOL * float(mx.max())
    assert float((tail - want).abs().max()) <= SNR_TOL * float(mx.max())
    assert float((j == am).float().mean()) > 0.99
