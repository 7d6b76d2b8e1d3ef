"""The strain windows that a bank keeps are those of the last closed tapes: tapes of
small calls do not keep larger ones out."""
import pytest

from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_kept_windows_follow_the_calls():
    from paper_1602_05573_amd import SpiirBank
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    bank = random_bank(108, 0, 1, 2, 2, 0.9, 0.99, 10)
    n = 1 << 24                       # a window of 64 MiB
    x = torch.from_numpy(strain(n, 108)).cuda()
    print("[case] kept windows", flush=True)

    def tape(bk, k):
        return bk.forward_z(x[:k].contiguous() if k < n else x, want_tape=True)

    with SpiirBank.from_bank(bank) as bk:
        small = [tape(bk, 100)[1], tape(bk, 200)[1]]
        for t in small:
            t.close()
        z, t = tape(bk, n)
        t.close()
        del z                         # back to the allocator, which the next call takes it from
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        z, t = tape(bk, n)
        torch.cuda.synchronize()
        taken = before - torch.cuda.mem_get_info()[0]
        t.close()
    assert taken < 32 << 20
