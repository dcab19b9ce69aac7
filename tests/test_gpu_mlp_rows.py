"""The network's kernels at batch sizes around their row groups and the sixteen
waves' shares of the batch, against the float64 reference; the bounds are
those of the other network tests (1e-5 for the forward pass and the loss, 1e-4
of an entry or of a quarter of its tensor's rms for gradients)."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 15, 17, 63, 257, 1000])
def test_forward_and_gradients_at_row_group_edges(B):
    import torch
    from paper_2208_09136_amd import rqa
    rng = np.random.default_rng(B)
    theta = (mlp.init(3) + rng.normal(0, 0.05, mlp.PARAMS)).astype(np.float32)
    X = rng.standard_normal((B, mlp.IN)).astype(np.float32)
    T = rng.standard_normal((B, mlp.OUT)).astype(np.float32)
    x, t = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    with rqa.Context(0, torch.cuda.current_stream()) as ctx:
        ctx.mlp_set_params(theta)
        y = torch.full((B + 1, mlp.OUT), 7.0, device="cuda")
        ctx.mlp_forward(x, y[:B])
        g, loss = ctx.mlp_gradients(x, t)
    assert torch.all(y[B] == 7.0)
    want, _ = mlp.forward(theta.astype(np.float64), X.astype(np.float64))
    assert np.max(np.abs(y[:B].cpu().numpy() - want) / (1.0 + np.abs(want))) < 1e-5
    L, grad = mlp.gradients(theta.astype(np.float64), X.astype(np.float64), T.astype(np.float64))
    assert abs(loss - L) <= 1e-5 * L
    got, ref = mlp.unpack(g.astype(np.float64)), mlp.unpack(grad)
    for name, _ in mlp.SIZES:
        s_t = np.sqrt(np.mean(ref[name] ** 2)) / 4
        assert np.all(np.abs(got[name] - ref[name]) <= 1e-4 * np.maximum(np.abs(ref[name]), s_t)), name
