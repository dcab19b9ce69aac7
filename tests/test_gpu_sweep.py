"""The threshold sweep around the target counts at which its histograms go from
64 to 32 columns and lose a workgroup per CU, counting both ranks (given
thresholds) and line ranks alone (after complete selection), against the
oracle."""
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


@pytest.mark.parametrize("lmin", [1, 2, 4])
@pytest.mark.parametrize("K", [1, 37, 38, 44, 45, 76, 77, 92, 93, 128])
def test_histogram_columns(ctx, K, lmin):
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(K)
    y = rng.standard_normal(901).astype(np.float32)
    rr = rng.permutation((np.arange(K) + 1) / K)
    rr[K // 2] = rr[0]  # one rate twice
    dev = torch.from_numpy(y).to("cuda:0")
    for m, tau, norm in ((1, 1, 0), (3, 5, 1), (2, 3, 0)):
        print(f"[sweep] K={K} lmin={lmin} m={m} tau={tau} norm={norm}", flush=True)
        want = oracle.run(y, m, tau, norm, 1, lmin, rr)
        got = ctx.run(dev, (m, tau, norm, 1, lmin), rr, rqa.RQA_SEL_PLAIN)
        curve = ctx.det_curve(dev, (m, tau, norm, 1, lmin), want["eps"])
        for out in (got, curve):
            assert np.array_equal(out["count"], want["count"])
            assert np.array_equal(out["rr"], want["rr"])
            assert np.array_equal(out["det"], want["det"], equal_nan=True)
        assert np.array_equal(got["eps"].view(np.uint32), want["eps"].view(np.uint32))


@pytest.mark.parametrize("norm,m,tau", [(0, 1, 1), (1, 3, 3), (1, 3, 5), (0, 4, 2)])
@pytest.mark.parametrize("lmin", range(3, 17))
def test_line_windows(ctx, lmin, norm, m, tau):
    # every split of lmin into window stages, diagonals and segments shorter
    # and longer than the window, against the oracle
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(lmin)
    for nv in (lmin, lmin + 1, 40, 64 + lmin, 129, 390):
        n = nv + (m - 1) * tau
        y = (np.sin(0.3 * np.arange(n)) + 0.1 * rng.standard_normal(n)).astype(np.float32)
        dev = torch.from_numpy(y).to("cuda:0")
        for K, w, segment in ((6, 1, 64), (6, 3, 320), (50, 1, 64)):
            if nv <= w:
                continue
            print(f"[windows] lmin={lmin} m={m} tau={tau} nv={nv} K={K} w={w}", flush=True)
            rr = np.linspace(0.05, 1.0, K)
            want = oracle.run(y, m, tau, norm, w, lmin, rr)
            ctx.set_shape(segment, 2)
            p = (m, tau, norm, w, lmin)
            for out in (ctx.run(dev, p, rr, rqa.RQA_SEL_PLAIN), ctx.run(dev, p, rr, rqa.RQA_SEL_SAMPLE),
                        ctx.det_curve(dev, p, want["eps"])):
                assert np.array_equal(out["count"], want["count"])
                assert np.array_equal(out["det"], want["det"], equal_nan=True)
            ctx.set_shape(0, 0)
