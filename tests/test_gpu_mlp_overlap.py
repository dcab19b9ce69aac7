"""The network's forward pass into memory that it also reads from: the output
starts at, inside, before or just past the input rows.  Results equal those
written elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

IN, OUT = 66, 20


# first output word, counted from the first input word, in rows of the batch
@pytest.mark.parametrize("at", ["start", "middle", "end", "past", "below", "before"])
@pytest.mark.parametrize("B", [1, 5, 4096])
def test_output_over_input(B, at):
    import torch
    from paper_2208_09136_amd import rqa
    first = {"start": 0, "middle": B * 30, "end": B * IN - 1, "past": B * IN, "below": -B * OUT + 1, "before": -B * OUT}[at]
    rng = np.random.default_rng(B)
    X = torch.from_numpy(rng.standard_normal((B, IN)).astype(np.float32)).cuda()
    memory = torch.full((B * (IN + 2 * OUT),), 7.0, device="cuda")
    lo = B * OUT
    x = memory[lo:lo + B * IN]
    y = memory[lo + first:lo + first + B * OUT]
    x.copy_(X.reshape(-1))
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        ctx.mlp_init(5)
        want = torch.empty(B, OUT, device="cuda")
        ctx.mlp_forward(X, want)
        expect = memory.clone()
        expect[lo + first:lo + first + B * OUT] = want.reshape(-1)
        print(f"[overlap] B={B} {at}", flush=True)
        ctx.mlp_forward(x, y)
    assert torch.equal(memory, expect)
