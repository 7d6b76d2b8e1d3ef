"""A captured backward goes on giving the same gradients after longer calls of the
bank have grown the adjoint scratch."""
import numpy as np
import pytest

from workloads import random_bank, strain

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_captured_backward_outlives_growth():
    from paper_1602_05573_amd import SpiirBank
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")
    bank = random_bank(109, 0, 3, 20, 20, 0.97, 0.9999, 300)
    rng = np.random.default_rng(109)

    def inputs(n):
        g = (rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))).astype(np.complex64)
        return torch.from_numpy(strain(n, 109)).cuda(), torch.from_numpy(g).cuda()

    print("[case] captured backward, scratch grown after it", flush=True)
    bk = SpiirBank.from_bank(bank)
    x, g = inputs(300)
    z, tape = bk.forward_z(x, want_tape=True)
    want = [v.clone() for v in bk.backward(tape, g)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ga, gb = bk.backward(tape, g, stream=side)
    held = []
    for n in (2000, 30000, 100000):
        xl, gl = inputs(n)
        zl, tl = bk.forward_z(xl, want_tape=True)
        first = [v.clone() for v in bk.backward(tl, gl)]
        held.append(torch.ones(1 << 18, device="cuda"))   # what freed scratch would be given to
        ga.zero_()
        gb.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ga, want[0]) and torch.equal(gb, want[1])
        assert all(bool((h == 1).all()) for h in held)
        assert all(torch.equal(a, b) for a, b in zip(bk.backward(tl, gl), first))
        torch.cuda.synchronize()
        tl.close()
    del graph
    tape.close()
    bk.close()
