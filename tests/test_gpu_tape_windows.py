"""Strain windows kept from closed tapes: forward and backward through windows of
other sizes and streams, a tape that outlives its bank, and a captured backward
give what fresh allocations give."""
import numpy as np
import pytest

import oracle
from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


def inputs(n, T, seed):
    rng = np.random.default_rng(seed)
    g = (rng.standard_normal((T, n)) + 1j * rng.standard_normal((T, n))).astype(np.complex64)
    return torch.from_numpy(strain(n, seed)).cuda(), torch.from_numpy(g).cuda()


def fresh(bank, x, g):
    from paper_1602_05573_amd import SpiirBank
    with SpiirBank.from_bank(bank) as bk:
        z, tape = bk.forward_z(x, want_tape=True)
        out = (z,) + tuple(bk.backward(tape, g))
        torch.cuda.synchronize()
        tape.close()
    return out


def test_windows_of_closed_tapes():
    from paper_1602_05573_amd import SpiirBank
    bank = random_bank(97, 0, 6, 10, 90, 0.97, 0.9999, 700)
    cases = [inputs(n, 6, 200 + n) for n in (3000, 900, 2900, 100, 3000, 4000)]
    want = [fresh(bank, x, g) for x, g in cases]
    print("[case] windows of closed tapes", flush=True)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    with SpiirBank.from_bank(bank) as bk:
        got = []
        for i, (x, g) in enumerate(cases * 3):   # the next call on another stream waits for the window alone
            s = streams[i % 3]
            s.wait_stream(streams[(i - 1) % 3])   # the bank's own scratch is one per bank
            with torch.cuda.stream(s):
                z, tape = bk.forward_z(x, want_tape=True)
                got.append((z,) + tuple(bk.backward(tape, g)))
                tape.close()
        torch.cuda.synchronize()
    for i, out in enumerate(got):
        for a, b in zip(out, want[i % len(cases)]):
            assert torch.equal(a, b)


def test_tape_outlives_bank_and_captured_backward():
    from paper_1602_05573_amd import SpiirBank
    bank = random_bank(98, 0, 3, 20, 20, 0.97, 0.9999, 300)
    x, g = inputs(1500, 3, 98)
    want = fresh(bank, x, g)
    print("[case] captured backward", flush=True)
    bk = SpiirBank.from_bank(bank)
    z, tape = bk.forward_z(x, want_tape=True)
    bk.backward(tape, g)   # grows the scratch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ga, gb = bk.backward(tape, g, stream=side)
    for _ in range(3):
        ga.zero_()
        gb.zero_()
        graph.replay()
        # another tape while the graph holds the first one's window
        z2, t2 = bk.forward_z(x * 2, want_tape=True)
        torch.cuda.synchronize()
        t2.close()
        assert torch.equal(ga, want[1]) and torch.equal(gb, want[2])
    del graph
    bk.close()
    tape.close()
