"""Launch shapes whose chunks hold more than 2^32 cells, on series of more than
2^32 pairs: the counters of a workgroup are 32-bit words, and every count must
still come out exact (shapes never change results).  The expected values are
the number of pairs itself, or those of the default shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE = (65536, 4096)  # the largest a caller may set: 2^34 cells per chunk


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2208_09136_amd import rqa
    c = rqa.Context(0, torch.cuda.current_stream())
    yield c
    c.close()


def pairs(n):
    return n * (n - 1) // 2


def test_given_thresholds(ctx):
    # every pair recurs, on one line per diagonal: one rank takes all cells
    import torch
    n = 93_000
    dev = torch.from_numpy(np.random.default_rng(3).standard_normal(n).astype(np.float32)).cuda()
    eps = np.array([1e6], np.float32)
    want = ctx.det_curve(dev, (1, 1, 0, 1, 2), eps)
    ctx.set_shape(*SHAPE)
    got = ctx.det_curve(dev, (1, 1, 0, 1, 2), eps)
    ctx.set_shape(0, 0)
    print("[cells] curve", got["count"], got["det"], flush=True)
    assert pairs(n) > 2 ** 32
    assert int(got["count"][0]) == pairs(n) and got["rr"][0] == 1.0
    assert got["det"][0] == (pairs(n) - 1) / pairs(n)  # the last diagonal is a single cell
    for k in ("count", "rr", "det"):
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("flag", ["RQA_SEL_PLAIN", "RQA_SEL_SAMPLE"])
@pytest.mark.parametrize("K", [3, 50])  # range sweep, threshold sweep after complete selection
def test_path(ctx, K, flag):
    # more than 2^32 line values below the first threshold
    import torch
    from paper_2208_09136_amd import rqa
    n = 95_000
    dev = torch.from_numpy(np.random.default_rng(4).standard_normal(n).astype(np.float32)).cuda()
    rr = np.linspace(0.97, 1.0, K)
    want = ctx.run(dev, (1, 1, 0, 1, 2), rr, getattr(rqa, flag))
    ctx.set_shape(*SHAPE)
    got = ctx.run(dev, (1, 1, 0, 1, 2), rr, getattr(rqa, flag))
    ctx.set_shape(0, 0)
    print(f"[cells] path K={K} {flag}", got["count"][-1], flush=True)
    assert int(got["count"][-1]) == pairs(n)
    assert got["det"][0] * int(got["count"][0]) > 2 ** 32
    for k in ("eps", "count", "det"):
        assert np.array_equal(got[k], want[k]), k


def test_one_key(ctx):
    # every key is 0: one bucket of the first selection pass takes all pairs
    import torch
    from paper_2208_09136_amd import rqa
    n = 93_000
    dev = torch.zeros(n, device="cuda")
    ctx.set_shape(*SHAPE)
    eps, k, count = ctx.select_thresholds(dev, (1, 1, 0, 1, 2), np.array([0.5, 1.0]), rqa.RQA_SEL_PLAIN)
    ctx.set_shape(0, 0)
    print("[cells] one key", count, flush=True)
    assert np.all(eps == 0.0) and np.all(count == pairs(n)) and int(k[1]) == pairs(n)
