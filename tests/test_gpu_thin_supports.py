"""Supports whose pixels share few flights run term by term: 600 pixels spread
over a 200 x 200 map (refused by their box) and 1000 over 150 x 150 (refused by
their records' rows); a disk of 1,000 pixels takes the flux stages.  Means against
the oracle (bar of the term-by-term path, 1e-4)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle as O  # noqa: E402
import synth  # noqa: E402


@pytest.mark.parametrize("nx,ny,n_p,launches", [(200, 200, 600, 1), (150, 150, 1000, 1), (40, 40, 0, 2)])
def test_route_and_means(nx, ny, n_p, launches):
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(2)
    mu = np.zeros(nx * ny, np.float32)
    if n_p:
        mu[rng.choice(nx * ny, n_p, replace=False)] = 0.2
    else:
        X, Y = synth.phantoms.pixel_centres(nx, ny, 0.2)
        mu[(np.hypot(X, Y) < 3.6).ravel()] = 0.2
    mu = mu.reshape(ny, nx)
    sup = np.flatnonzero(mu.ravel())
    assert len(sup) >= 512
    g = synth.Geometry(nx, ny, 0.2, 64, 0.25 * nx / 64, 8, fwhm_u_cm=0.5)
    ev = {"angle": rng.integers(0, 8, 300).astype(np.int32),
          "u_bin": rng.uniform(24.0, 40.0, 300).astype(np.float32),
          "energy": rng.uniform(100.0, 175.0, 300).astype(np.float32)}
    img = np.zeros(nx * ny, np.float32)
    q = np.sort(rng.choice(sup, 40, replace=False)).astype(np.int32)
    img[q] = rng.uniform(1.0, 3.0, 40)
    img = img.reshape(ny, nx)
    ref = O.OracleModel(g.as_dict(), mu).system_matrix(ev, q) @ img.ravel()[q].astype(np.float64)
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev))
    try:
        L.lmosem_set_timing(ctx.handle, True)
        got = ctx.forward(L.events_to_device(ev, dev), torch.as_tensor(img, device=dev)).cpu().numpy()
        assert ctx.stats()["forward_launches"] == launches
    finally:
        ctx.close()
    live = ref > 1e-8 * ref.max()
    assert live.sum() >= 200
    assert np.max(np.abs(got - ref)[live] / ref[live]) <= 1e-4
