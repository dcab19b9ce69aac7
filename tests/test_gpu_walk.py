"""The key walkers at the ends of diagonals: numbers of vectors around the band
width and the block lengths, compiled and run-time embeddings, component
counts around the unrolled four, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2208_09136_amd import rqa
    c = rqa.Context(0, torch.cuda.current_stream())
    yield c
    c.close()


@pytest.mark.parametrize("norm", [0, 1])
@pytest.mark.parametrize("m,tau", [(1, 1), (3, 3), (3, 5), (2, 7), (4, 1), (5, 3), (9, 2)])
def test_ends_of_diagonals(ctx, m, tau, norm):
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(m * 100 + tau)
    rr = np.array([0.05, 0.2, 0.5, 1.0])
    for nv in (2, 3, 17, 63, 64, 65, 66, 81, 96, 127, 129, 191, 200, 333):
        for w, lmin in ((1, 2), (1, 1), (5, 2)):
            if nv <= w:
                continue
            y = rng.standard_normal(nv + (m - 1) * tau).astype(np.float32)
            print(f"[walk] m={m} tau={tau} norm={norm} nv={nv} w={w} lmin={lmin}", flush=True)
            want = oracle.run(y, m, tau, norm, w, lmin, rr)
            lines = oracle.lines(y, m, tau, norm, w, lmin, want["eps"], hist_len=nv + 1)
            dev = torch.from_numpy(y).to("cuda:0")
            offs = np.array([0, len(y)], np.uint64)
            for segment in (64, 192):
                ctx.set_shape(segment, 2)
                for flags in (rqa.RQA_SEL_PLAIN, rqa.RQA_SEL_SAMPLE):
                    got = ctx.run(dev, (m, tau, norm, w, lmin), rr, flags)
                    assert np.array_equal(got["eps"].view(np.uint32), want["eps"].view(np.uint32))
                    assert np.array_equal(got["count"], want["count"])
                    assert np.array_equal(got["det"], want["det"], equal_nan=True)
                full = ctx.batch_hist(dev, offs, [(m, tau, norm, w, lmin)], rr[None], nv + 1)
                assert np.array_equal(full["hist"][0], lines["hist"])
                curve = ctx.det_curve(dev, (m, tau, norm, w, lmin), want["eps"])
                assert np.array_equal(curve["count"], want["count"]) and np.array_equal(curve["det"], want["det"], equal_nan=True)
                thresholds = ctx.select_thresholds(dev, (m, tau, norm, w, lmin), rr)[0]
                assert np.array_equal(thresholds.view(np.uint32), want["eps"].view(np.uint32))
            ctx.set_shape(0, 0)
