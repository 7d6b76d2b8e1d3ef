"""Fused max / argmax of banks whose templates are cut into parts: the keys of
slices of split templates give the maximum of the stored rows, bit for bit, with
split counts around the slice length, beside whole templates, in every piece of a call."""
import numpy as np
import pytest

from workloads import Bank, random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


def check(bank, cuts, want_split, **opts):
    from paper_1602_05573_amd import SpiirBank
    x = torch.from_numpy(strain(cuts[-1], 102)).cuda()
    with SpiirBank.from_bank(bank, **opts) as bk:
        assert (bk.info["n_parts"] > 0) == (want_split > 0)
        rows = torch.cat([bk.filter_block(x[a:b].contiguous()) for a, b in zip(cuts[:-1], cuts[1:])], dim=1)
        for noalloc in (False, True):
            bk.reset()
            mx, am = [], []
            for a, b in zip(cuts[:-1], cuts[1:]):
                out = (torch.empty(b - a, device="cuda"), torch.empty(b - a, dtype=torch.int32, device="cuda"))
                (bk.trigger_max_noalloc if noalloc else bk.trigger_max)(x[a:b].contiguous(), out=out)
                mx.append(out[0])
                am.append(out[1])
            top = rows.max(dim=0).values
            assert torch.equal(torch.cat(mx), top)
            first = (rows == top[None, :]).to(torch.int32).argmax(dim=0).to(torch.int32)
            assert torch.equal(torch.cat(am), first)


@pytest.mark.parametrize("n_split", [1, 7, 8, 9, 130])
def test_keys_of_split_templates(n_split):
    """Templates of two delays in different bands beside templates of one."""
    rng = np.random.default_rng(n_split)
    bank = random_bank(102, n_split, n_split + 5, 3, 20, 0.99, 0.999, 500)
    d = (bank.d % 100).astype(np.int32)
    for j in rng.permutation(n_split + 5)[:n_split]:
        d[int(bank.offsets[j + 1]) - 1] += 300
    print("[case] keys of %d split templates" % n_split, flush=True)
    check(Bank(bank.offsets, bank.a, bank.b, d, 500), [0, 1, 64, 1000], n_split, delay_band=256, max_block=512,
          time_split=1)


def test_keys_of_automatic_bands():
    bank = random_bank(103, 0, 90, 380, 420, 0.99, 1 - 1e-5, 60000)
    print("[case] keys of automatic bands", flush=True)
    check(bank, [0, 64, 700, 5000], 90)
