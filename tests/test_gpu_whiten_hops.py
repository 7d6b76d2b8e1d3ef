"""The whitening transforms at every frame length, at the edges of a call: one
hop, an even number of max_block pieces, frame pairs with one frame, an output
that is the input, a captured call, samples that are not finite."""
import numpy as np
import pytest

import oracle
from workloads import coloured_noise

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-4   # of the largest value, the gate of the other whitening tests


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU test run without a GPU")


@pytest.mark.parametrize("N", [1 << k for k in range(4, 14)])
def test_every_frame_length(N):
    from paper_1602_05573_amd import Whitener
    H = N // 2
    x = coloured_noise(17 * H, 7)
    print("[case] hops N=%d" % N, flush=True)
    xd = torch.from_numpy(x).cuda()
    with Whitener(N, max_block=4 * H) as wh:
        for frames in (8, 1, 7):   # pairs of frames, one frame alone, a pair with one frame
            t = x[:(frames + 1) * H + (H - 1 if frames == 7 else 0)]
            wh.estimate_psd(torch.from_numpy(t.copy()).cuda())
            S = oracle.welch_psd(t, N)
            assert np.max(np.abs(wh.psd() - S)) <= TOL * S.max()
        wh.estimate_psd(xd)
        S = wh.psd()
        # 1 hop, pieces of 4 hops: 2 (even), 1 with a rest, 1, then in place over 2 pieces
        cuts = [0, 1, 9, 10, 17]
        got = [wh.process(xd[a * H:b * H].clone()) for a, b in zip(cuts[:-2], cuts[1:-1])]
        last = xd[10 * H:].clone()
        got.append(wh.process(last, out=last))
        more = wh.process(xd[:H].clone())
    ref = oracle.whiten(np.concatenate([x, x[:H]]), S, N)
    got = torch.cat(got + [more]).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref))


def test_captured_call_of_two_pieces():
    """The stored half frames are where the replays of a captured call of an
    even number of pieces take them from."""
    from paper_1602_05573_amd import Whitener
    N, H = 256, 128
    x = coloured_noise(8 * 4 * H, 8)
    print("[case] captured whitening", flush=True)
    with Whitener(N, max_block=2 * H) as wh:
        wh.set_psd(np.ones(H + 1))
        xin = torch.from_numpy(x[:4 * H].copy()).cuda()
        out = torch.zeros_like(xin)
        got = [wh.process(xin).cpu()]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            wh.process(xin, out=out, stream=side)
        for i in range(1, 8):
            xin.copy_(torch.from_numpy(x[4 * i * H:4 * (i + 1) * H].copy()))
            graph.replay()
            torch.cuda.synchronize()
            got.append(out.cpu())
    ref = oracle.whiten(x, np.ones(H + 1), N)
    assert np.max(np.abs(torch.cat(got).numpy() - ref)) <= TOL * np.max(np.abs(ref))


def test_samples_not_finite_stay_in_their_frames():
    from paper_1602_05573_amd import Whitener
    N, H = 64, 32
    x = coloured_noise(8 * H, 9)
    x[3 * H + 5] = np.nan
    print("[case] not finite", flush=True)
    with Whitener(N) as wh:
        wh.set_psd(np.ones(H + 1))
        xd = torch.from_numpy(x).cuda()
        # the second call has one frame with the sample, then one without
        got = torch.cat([wh.process(xd[:4 * H].clone()), wh.process(xd[4 * H:6 * H].clone()),
                         wh.process(xd[6 * H:].clone())]).cpu().numpy()
    # sample 3H+5 is in frames 3 and 4 (hops 3..5 hold a half of one of them)
    bad = np.isnan(got).reshape(8, H).all(axis=1)
    assert bad.tolist() == [False, False, False, True, True, True, False, False]
    assert np.isfinite(got[:3 * H]).all() and np.isfinite(got[6 * H:]).all()
