"""Selection and sweeps on series of few distinct values, where from two to all
lanes of a wave add to the same counters, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flag", ["RQA_SEL_PLAIN", "RQA_SEL_SAMPLE"])
@pytest.mark.parametrize("K", [1, 3, 20, 60])
@pytest.mark.parametrize("values", [2, 20, 300, 5000])
def test_tied_keys(values, K, flag):
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(values)
    y = (rng.integers(0, values, 700) / 16.0).astype(np.float32)
    rr = (np.arange(K) + 1) / (2.0 * K)
    dev = torch.from_numpy(y).cuda()
    print(f"[ties] {values} K={K} {flag}", flush=True)
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        for p in ((1, 1, 0, 1, 2), (2, 3, 1, 4, 3)):
            want = oracle.run(y, *p, rr)
            eps, k, count = ctx.select_thresholds(dev, p, rr, getattr(rqa, flag))
            got = ctx.run(dev, p, rr, getattr(rqa, flag))
            assert np.array_equal(eps, want["eps"]) and np.array_equal(count, want["count"])
            for key in ("eps", "count", "det"):
                assert np.array_equal(got[key], want[key], equal_nan=True), key
