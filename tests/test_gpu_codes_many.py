"""The range sweep's code table at the most targets that take it (44 with plain
selection, 40 with a window; more take complete selection and the threshold
sweep): many groups sharing buckets, high odd codes, 32-column rows, on the edge
signals of the code-table tests, against the oracle.  The number of full passes
says that the range sweep ran."""
import numpy as np
import pytest

import oracle
from test_gpu_codes import series

pytestmark = pytest.mark.gpu

# full passes: two counting passes and the range sweep; a window pass and the
# range sweep, then the plain passes for a target outside the window
PATHS = {"RQA_SEL_PLAIN": (44, (3,)), "RQA_SEL_SAMPLE": (40, (2, 5))}


@pytest.mark.parametrize("flag", sorted(PATHS))
@pytest.mark.parametrize("kind", ["decades", "ties", "near_equal", "noise"])
@pytest.mark.parametrize("m,tau,norm,lmin", [(1, 1, 0, 2), (3, 5, 1, 2), (3, 3, 1, 1), (2, 2, 1, 3)])
def test_most_targets(kind, flag, m, tau, norm, lmin):
    import torch
    from paper_2208_09136_amd import rqa
    K, passes = PATHS[flag]
    y = series(kind, 421)
    dev = torch.from_numpy(y).to("cuda:0")
    p = (m, tau, norm, 1, lmin)
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        for rr in ((np.arange(K) + 1) / K, 0.3 + 1e-4 * np.arange(K), (np.arange(K) + 1) / 1000.0):
            print(f"[codes] {kind} {flag} {p} {rr[0]}", flush=True)
            want = oracle.run(y, *p, rr)
            got = ctx.run(dev, p, rr, getattr(rqa, flag))
            assert ctx.selection_stats()["full_passes"] in passes
            assert np.array_equal(got["eps"].view(np.uint32), want["eps"].view(np.uint32))
            assert np.array_equal(got["count"], want["count"])
            assert np.array_equal(got["det"], want["det"], equal_nan=True)
        more = (np.arange(K + 1) + 1) / (K + 1)
        ctx.run(dev, p, more, getattr(rqa, flag))
        assert ctx.selection_stats()["full_passes"] == (4 if flag == "RQA_SEL_PLAIN" else
                                                        3 + 3 * (ctx.selection_stats()["series_fallback"] > 0))
