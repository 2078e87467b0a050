"""Tables of direction terms whose entries are the pixel offsets of the
support's bounding box or, where that has more of them than the support has
pairs, the pairs themselves: binned rows and the path table with either, formed
in one run of angles and in several, against FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle as O  # noqa: E402
import synth  # noqa: E402


# support pixels spread over a 200 x 203 map, energy bins: 161,595 offsets
# against 6,400, 90,000 and 202,500 pairs; 32 angles in 1, 2 and 2 runs
@pytest.mark.parametrize("n_p,edges", [(80, [100.0, 143.0, 175.0]),
                                       (300, [100.0, 120.0, 130.0, 143.0, 175.0]),
                                       (450, [100.0, 130.0, 175.0])])
def test_binned_rows_of_spread_supports(n_p, edges):
    """Three iterations of binned OS-MLEM against FP64 EM on the per-bin
    kernel's rows: both rows are FP64 sums rounded to FP32 (6e-8), and means and
    backprojections sum at most 450 and 1,280 FP32 products, whose roundings
    add as their square root: 12 sub-iterations of sqrt(1,730) * 6e-8 each,
    3e-5."""
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    g = synth.Geometry(200, 203, 0.1, 160, 0.15, 32, fwhm_u_cm=0.4, n_subsets=4).as_dict()
    rng = np.random.default_rng(5)
    mu = np.zeros(200 * 203, np.float32)
    sup = np.sort(rng.choice(200 * 203, n_p, replace=False))
    sup[0], sup[-1] = 0, 200 * 203 - 1   # the box is the whole map
    mu[sup] = rng.uniform(0.1, 0.3, n_p).astype(np.float32)
    mu = mu.reshape(203, 200)
    n_pos, n_e = 40, len(edges) - 1
    n_bins = 32 * n_pos * n_e
    y = rng.integers(1, 5, size=n_bins).astype(np.float32)
    ctx = L.Context(g, torch.as_tensor(mu, device=dev))
    try:
        rows = torch.empty((n_bins, 203, 200), device=dev)
        L.lmosem_binned_rows(ctx.handle, n_pos, edges, torch.arange(n_bins, dtype=torch.int32, device=dev), rows)
        H = rows.reshape(n_bins, -1)[:, torch.as_tensor(sup, device=dev)].cpu().numpy().astype(np.float64)
        del rows
        y[H.sum(1) == 0] = 0
        img = torch.empty((203, 200), device=dev)
        L.lmosem_binned_reconstruct(ctx.handle, n_pos, edges, torch.as_tensor(y, device=dev), 3, img)
        got = img.cpu().numpy().ravel()
    finally:
        ctx.close()
    assert (H.sum(1) > 0).sum() > 500
    ref = O.binned_os_mlem(H, y.astype(np.float64), np.repeat(np.arange(32), n_pos * n_e), 4, 3, np.ones(n_p))
    assert np.all(np.delete(got, sup) == 0)
    err = np.abs(got[sup] - ref)
    tol = np.where(ref >= 1e-2 * ref.max(), 3e-5 * ref, 3e-7 * ref.max())
    assert np.all(err <= tol), float(np.max(err / np.maximum(ref, 1e-300)))


# 1,436 support pixels and an emission set of 1 pixel (its pairs are fewer than
# the box's 7,469 offsets) or of some fifty (500 angles' terms: 75 MB, two runs)
@pytest.mark.parametrize("radius,n_angles", [(0.1, 40), (1.6, 500)])
def test_path_table_of_small_emission_sets(radius, n_angles):
    """Two iterations of 300 events, which go term by term, against the oracle
    (bar of the term-by-term path, 1e-4 a mean)."""
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    _, mu = synth.phantom(synth.workload("brain64"))
    X, Y = synth.phantoms.pixel_centres(64, 64, 0.4)
    mask = (mu > 0) & (np.hypot(X - 1.8, Y - 1.4) <= radius)
    assert (mu > 0).sum() == 1436 and mask.sum() in ([1] if radius < 1 else range(45, 60))
    g = synth.Geometry(64, 64, 0.4, 128, 0.2, n_angles)
    ev = synth.generate_events(g, mask.astype(np.float32), mu, 300, 4)
    ev = {k: ev[k] for k in ("angle", "u_bin", "energy")}
    m = O.OracleModel(g.as_dict(), mu)
    q = np.flatnonzero(mask.ravel()).astype(np.int32)
    img = torch.as_tensor(mask.astype(np.float32), device=dev).contiguous()
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev),
                    emission=torch.as_tensor(mask.astype(np.float32), device=dev))
    try:
        sens = ctx.sensitivity(-1).cpu().numpy().ravel()[q].astype(np.float64)
        evs = L.lmosem_events_load(ctx.handle, L.events_to_device(ev, dev))
        try:
            L.lmosem_set_timing(ctx.handle, True)
            L.lmosem_iterate(ctx.handle, evs, 2, img)
            torch.cuda.synchronize()
            assert ctx.stats()["forward_launches"] == 2   # (one a sub-iteration: term by term)
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()
    H, f = m.system_matrix(ev, q), np.ones(len(q))
    for _ in range(2):
        mean = H @ f
        f = f * (H.T @ np.where(mean > 1e-30, 1.0 / np.maximum(mean, 1e-30), 0.0)) / sens
    got = img.cpu().numpy().ravel()[q]
    assert np.max(np.abs(got - f) / np.maximum(f, 1e-3 * f.max())) <= 1e-4
