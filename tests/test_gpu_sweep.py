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
