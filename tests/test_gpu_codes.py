"""The range sweep's code table at its edges, against the oracle: groups that
share a bucket, groups at key 0 and at +inf, one group, many close groups,
tied keys, every line class, plain and windowed candidate ranges."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2208_09136_amd import rqa
    c = rqa.Context(0, torch.cuda.current_stream())
    yield c
    c.close()


def series(kind, n):
    rng = np.random.default_rng(17)
    if kind == "decades":       # keys from denormals to +inf: the table's widest span
        return (rng.choice([-1.0, 1.0], n) * 10.0 ** rng.uniform(-25, 25, n)).astype(np.float32)
    if kind == "ties":          # few distinct keys, so most values have odd codes
        return rng.integers(0, 5, n).astype(np.float32)
    if kind == "near_equal":    # every key within a few patterns of its neighbours
        return (1.0 + rng.integers(0, 40, n) * 2.0 ** -23).astype(np.float32)
    return synth.series("logistic", n, 5.0, (17, 1, 0, 0))


TARGETS = {"one": [0.4], "close": [0.3 + 1e-6 * i for i in range(16)], "ends": [1e-9, 0.5, 1.0],
           "many": [(i + 1) / 64 for i in range(64)]}


@pytest.mark.parametrize("targets", sorted(TARGETS))
@pytest.mark.parametrize("kind", ["decades", "ties", "near_equal", "noise"])
@pytest.mark.parametrize("m,tau,norm,lmin", [(1, 1, 0, 2), (3, 5, 1, 2), (3, 3, 1, 1), (2, 2, 1, 3)])
def test_code_table_edges(ctx, kind, targets, m, tau, norm, lmin):
    from paper_2208_09136_amd import rqa
    import torch
    y = series(kind, 421)
    rr = np.array(TARGETS[targets])
    print(f"[codes] {kind} {targets} m={m} tau={tau} norm={norm} lmin={lmin}", flush=True)
    want = oracle.run(y, m, tau, norm, 1, lmin, rr)
    dev = torch.from_numpy(y).to("cuda:0")
    for flags in (rqa.RQA_SEL_PLAIN, rqa.RQA_SEL_SAMPLE):
        got = ctx.run(dev, (m, tau, norm, 1, lmin), rr, flags)
        assert np.array_equal(got["eps"].view(np.uint32), want["eps"].view(np.uint32))
        assert np.array_equal(got["count"], want["count"])
        assert np.array_equal(got["det"], want["det"], equal_nan=True)
