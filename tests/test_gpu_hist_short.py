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
