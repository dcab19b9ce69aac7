"""Batches of very many kernel variants (norm, embedding class, line class):
each variant is a launch of its own in every phase, the second and later ones on
a second stream, and a call's launches are limited.  A call over the limit is
refused as a whole, before its first launch, and leaves the next one alone."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

VARIANTS = [(m, tau, norm, 1, lmin) for norm in (0, 1) for m, tau in ((1, 1), (3, 3), (3, 5), (2, 2))
            for lmin in range(1, 17)]
LIMIT = 256  # work-queue counters, one per launch


def batch(count, seed):
    rng = np.random.default_rng(seed)
    ys = [rng.standard_normal(150 + i % 7).astype(np.float32) for i in range(count)]
    offsets = np.cumsum([0] + [len(y) for y in ys]).astype(np.uint64)
    return ys, np.concatenate(ys), offsets, VARIANTS[:count]


# launches per variant: plain selection three (two passes and the range sweep),
# the sample window two
@pytest.mark.parametrize("flag,per", [("RQA_SEL_PLAIN", 3), ("RQA_SEL_SAMPLE", 2)])
def test_up_to_the_limit(flag, per):
    import torch
    from paper_2208_09136_amd import rqa
    rr = np.array([0.05, 0.3])
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        most = LIMIT // per
        if most < len(VARIANTS):
            _, y, offsets, p = batch(most + 1, 1)
            print(f"[variants] {flag} {most + 1}", flush=True)
            with pytest.raises(rqa.RqaError) as e:
                ctx.batch(torch.from_numpy(y).cuda(), offsets, p, np.tile(rr, (len(p), 1)), getattr(rqa, flag))
            assert e.value.name == "RQA_ERR_UNSUPPORTED"
        ys, y, offsets, p = batch(min(most, len(VARIANTS)), 2)
        print(f"[variants] {flag} {len(p)}", flush=True)
        got = ctx.batch(torch.from_numpy(y).cuda(), offsets, p, np.tile(rr, (len(p), 1)), getattr(rqa, flag))
        for s, (series, (m, tau, norm, w, lmin)) in enumerate(zip(ys, p)):
            want = oracle.run(series, m, tau, norm, w, lmin, rr)
            assert np.array_equal(got["eps"][s].view(np.uint32), want["eps"].view(np.uint32)), s
            assert np.array_equal(got["count"][s], want["count"]), s
            assert np.array_equal(got["det"][s], want["det"], equal_nan=True), s
