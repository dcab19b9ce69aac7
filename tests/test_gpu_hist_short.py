"""Line histograms of few entries per row, whose last entry takes most lines:
rows around the 64 lengths that are counted in LDS, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,tau,norm", [(1, 1, 0), (3, 5, 1)])
@pytest.mark.parametrize("hist_len", [1, 2, 16, 63, 64, 65, 66, 700])
def test_row_lengths(hist_len, m, tau, norm):
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(hist_len)
    n = 640
    y = (np.sin(0.05 * np.arange(n)) + 0.02 * rng.standard_normal(n)).astype(np.float32)  # lines of every length
    eps = oracle.select(y, m, tau, norm, 1, np.array([0.02, 0.1, 0.4, 0.9, 1.0]))[0]
    dev = torch.from_numpy(y).cuda()
    print(f"[short] hist_len={hist_len} m={m}", flush=True)
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        for w, segment in ((1, 0), (7, 64), (1, 320)):
            ctx.set_shape(segment, 0)
            got = ctx.det_curve(dev, (m, tau, norm, w, 2), eps, hist_len=hist_len)
            want = oracle.lines(y, m, tau, norm, w, 2, eps, hist_len=hist_len)
            assert np.array_equal(got["hist"], want["hist"]), (w, segment)
            assert np.array_equal(got["det"], want["det"])


@pytest.mark.parametrize("kind", ["sine", "constant", "staircase", "two_values"])
@pytest.mark.parametrize("n", [64, 1500])
def test_runs_of_one_rank(kind, n):
    # neighbouring cells of equal rank, across blocks, full lists and segments
    import torch
    from paper_2208_09136_amd import rqa
    t = np.arange(n)
    y = {"sine": np.sin(2 * np.pi / 37.3 * t), "constant": 0 * t, "staircase": np.floor(t / 13) % 17,
         "two_values": (t // 9) % 2}[kind].astype(np.float32)
    dev = torch.from_numpy(y).cuda()
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        for p in ((1, 1, 0, 1, 2), (3, 3, 1, 2, 2), (2, 2, 0, 1, 2)):
            eps = np.sort(np.concatenate([oracle.select(y, *p[:4], np.linspace(0.05, 1.0, 9))[0], [0.0, 0.5, 50.0]]))
            want = oracle.lines(y, *p, eps.astype(np.float32), hist_len=n + 1)["hist"]
            for segment in (0, 64, 1024):
                print(f"[runs] {kind} n={n} {p} segment={segment}", flush=True)
                ctx.set_shape(segment, 0)
                got = ctx.det_curve(dev, p, eps, hist_len=n + 1)["hist"]
                ctx.set_shape(0, 0)
                assert np.array_equal(got, want)
