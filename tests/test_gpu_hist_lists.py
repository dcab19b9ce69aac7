"""The histogram pass's per-lane lists and stacks at their limits: one to 32
thresholds, segments shorter and longer than the range of a list's positions,
rows of one entry up to the longest line, on signals with many short lines, few
recurrent cells and runs through whole segments, against the oracle."""
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


def signal(kind, n):
    rng = np.random.default_rng(n)
    noise = rng.standard_normal(n)
    if kind == "sine":
        noise = np.sin(2 * np.pi / 37.3 * np.arange(n)) + 0.05 * noise
    elif kind == "steps":  # constant stretches: ties and runs through segments
        noise = np.round(np.repeat(noise, 200)[:n] * 2)
    return noise.astype(np.float32)


@pytest.mark.parametrize("kind,low", [("noise", 0.0), ("noise", 0.9), ("sine", 0.0), ("steps", 0.0)])
@pytest.mark.parametrize("K", [1, 2, 31, 32])
def test_lists(ctx, K, kind, low):
    import torch
    for n, m, tau, norm in ((2500, 1, 1, 0), (2301, 3, 5, 1)):
        y = signal(kind, n)
        rr = 0.001 + low + (0.999 - low) * np.arange(1, K + 1) / K if low else 0.002 * np.arange(1, K + 1)
        eps = oracle.select(y, m, tau, norm, 1, rr)[0]
        nv = n - (m - 1) * tau
        want = oracle.lines(y, m, tau, norm, 1, 2, eps, hist_len=nv + 1)["hist"]
        dev = torch.from_numpy(y).to("cuda:0")
        for segment, rows in ((0, nv + 1), (64, 1), (448, 65), (2176, 40)):
            print(f"[lists] {kind} K={K} low={low} n={n} m={m} segment={segment} rows={rows}", flush=True)
            ctx.set_shape(segment, 0)
            got = ctx.det_curve(dev, (m, tau, norm, 1, 2), eps, 2, rows)["hist"]
            ctx.set_shape(0, 0)
            ref = want[:, :rows].copy()
            ref[:, -1] += want[:, rows:].sum(1).astype(ref.dtype)  # the last entry holds all longer lines
            assert np.array_equal(got, ref)


@pytest.mark.parametrize("S,K", [(3, 32), (24, 32), (70, 9)])
def test_rows_of_a_batch(ctx, S, K):
    # lines shorter and longer than the lengths that fit the pinned staging,
    # next to series that have short ones only
    import torch
    ys = [signal(("noise", "steps", "sine")[i % 3], 300 + 1000 * ((7 * i) % S) // S) for i in range(S)]
    offs = np.concatenate([[0], np.cumsum([len(y) for y in ys])]).astype(np.uint64)
    prm = [(1, 1, 0, 1, 2) if i % 2 else (3, 5, 1, 1, 2) for i in range(S)]
    rr = np.tile(np.linspace(0.01, 0.4, K), (S, 1))
    dev = torch.from_numpy(np.concatenate(ys)).to("cuda:0")
    for rows in (1301, 129, 64):
        print(f"[rows] S={S} K={K} rows={rows}", flush=True)
        got = ctx.batch_hist(dev, offs, prm, rr, rows)
        for i, y in enumerate(ys):
            want = oracle.lines(y, *prm[i], got["eps"][i], hist_len=rows)["hist"]
            assert np.array_equal(got["hist"][i], want), i
