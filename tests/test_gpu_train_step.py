"""GPU tests of the training step's kernels at the sizes where they can go
wrong: one workgroup's 16 samples, slices of the weight gradients that do not
divide the batch, and more samples than the largest number of slices takes at
256 each; outputs, gradients and a training step agree on every size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import mlp as M  # noqa: E402
import synth  # noqa: E402


@pytest.mark.parametrize("count", [16, 528, 8208])
def test_step_sizes_match_reference(count):
    """Against the FP64 reference that rounds to bf16 at the same points: the
    bounds are the ones of the sizes in between (2e-3 of each array's largest
    entry: FP32 against FP64 sums, and a bf16 delta's last bit at a rounding
    tie, 2^-8 of one sample's share, which for 16 samples is at most 2^-8 / 16
    of a sum of entries of one size, doubled)."""
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    p = synth.mlp_init_params(5)
    rng = np.random.default_rng(count)
    X = rng.normal(size=(count, 8)).astype(np.float32)
    dy = rng.normal(size=count).astype(np.float32) / count
    t = rng.normal(size=count).astype(np.float32)
    net = L.lmosem_net_create(p)
    try:
        Xd = torch.as_tensor(X, device=dev)
        y = torch.empty(count, device=dev)
        L.lmosem_net_forward_train(net, Xd, y)
        got_y = y.cpu().numpy().astype(np.float64)
        g = L.lmosem_net_gradient(net, Xd, torch.as_tensor(dy, device=dev))
        loss = L.lmosem_net_train(net, Xd, torch.as_tensor(t, device=dev), batch=count, epochs=1, lr=1e-3)
    finally:
        L.lmosem_net_destroy(net)
    ref_y, cache = M.forward(p, X, bf16_round=True)
    ref = M.backward(p, cache, dy, bf16_round=True)
    assert np.max(np.abs(got_y - ref_y)) <= 2e-3 * max(1.0, np.max(np.abs(ref_y)))
    for k in ref:
        r, gk = ref[k].ravel(), g[k].ravel().astype(np.float64)
        assert np.max(np.abs(gk - r)) <= 2e-3 * max(float(np.max(np.abs(r))), 1e-30), k
    # the step's loss: the mean of squared FP32 differences, added in FP64
    mse = float(np.mean((got_y - t) ** 2))
    assert abs(float(np.ravel(loss)[0]) - mse) <= 1e-6 * mse
