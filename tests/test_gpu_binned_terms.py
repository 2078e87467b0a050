"""GPU tests of the all-bins rows with the direction terms tabulated by pixel
offset, where the table holds only some of the angles at a time (a wide map),
against rows evaluated path by path."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle as O  # noqa: E402
import synth  # noqa: E402


@pytest.mark.parametrize("scatter", [0, 1])
@pytest.mark.parametrize("edges", [[100.0, 175.0], [100.0, 125.0, 143.0, 175.0], [100.0, 120.0, 130.0, 143.0, 175.0]])
def test_wide_map_rows_match_per_path_rows(edges, scatter):
    """A 200 x 203 map with a small off-centre support: 2.6 MB of terms per
    angle and energy bin, so that 32 angles take several rounds; 3 iterations
    of binned OS-MLEM against FP64 EM on the per-bin kernel's rows.  Both rows
    are FP64 sums rounded to FP32 (6e-8); means and backprojections sum at most
    77 and 128 FP32 products, so 3 iterations of 4 subsets stay within some
    12 * (77 + 128) * 6e-8 = 1.5e-4."""
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    g = synth.Geometry(200, 203, 0.4, 160, 0.6, 32, n_subsets=4).as_dict()
    g = dict(g, scatter_model=scatter)
    mu = np.zeros((203, 200), np.float32)
    mu[120:127, 60:71] = 0.15
    mu[122, 64] = 0.3
    n_pos, n_e = 40, len(edges) - 1
    rng = np.random.default_rng(3)
    y = rng.integers(0, 4, size=32 * n_pos * n_e).astype(np.float32)
    ctx = L.Context(g, torch.as_tensor(mu, device=dev))
    try:
        sup = np.flatnonzero(mu.ravel() > 0)
        rows = torch.empty((32 * n_pos * n_e, 203, 200), device=dev)
        L.lmosem_binned_rows(ctx.handle, n_pos, edges,
                             torch.arange(32 * n_pos * n_e, dtype=torch.int32, device=dev), rows)
        H = rows.cpu().numpy().reshape(len(y), -1)[:, sup].astype(np.float64)
        del rows
        y[H.sum(1) == 0] = 0
        img = torch.empty((203, 200), device=dev)
        L.lmosem_binned_reconstruct(ctx.handle, n_pos, edges, torch.as_tensor(y, device=dev), 3, img)
        got = img.cpu().numpy().ravel()
    finally:
        ctx.close()
    assert (H.sum(1) > 0).sum() > 100
    ref = O.binned_os_mlem(H, y.astype(np.float64), np.repeat(np.arange(32), n_pos * n_e), 4, 3, np.ones(len(sup)))
    assert np.all(np.delete(got, sup) == 0)
    err = np.abs(got[sup] - ref)
    tol = np.where(ref >= 1e-2 * ref.max(), 1.5e-4 * ref, 1.5e-6 * ref.max())
    assert np.all(err <= tol), float(np.max(err / np.maximum(ref, 1e-300)))
