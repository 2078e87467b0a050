"""Sub-iterations through directional flux (the stages that replace the
term-by-term kernels once a sub-iteration has enough events) against the FP64
oracle, at the sizes where their tiles, sectors and blocks end: odd grids,
partial blocks of pixels and events, empty angles, few and many direction and
energy nodes, emission sets, several realisations.

Tolerances: a path's interpolation error is at most 5e-7 in energy and, in
direction, 2e-6 within six widths of the energy response and 5e-5 within
eight; FP32 sums add about 1e-6.  Events beyond six widths of every path that
reaches them hardly occur, so means are held to 2e-5 (1e-4, the bar of the
term-by-term path, for masked emission, where they do) and sums over many
events to 5e-6."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle as O  # noqa: E402
import synth  # noqa: E402


def _lib():
    from paper_2002_12471_amd import lmosem as L
    return L


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available()
    return torch.device("cuda:0")


# (grid, angles, subsets, energy FWHM, window, events, scatter): the event
# counts put every case above the rule's threshold; a narrow response needs
# many nodes, a wide one the fewest; 3 empty angles in the second case
CASES = {
    "disk16": (16, 16, 1, 15.9, (100.0, 175.0), 400_000, 1),
    "odd21": (21, 17, 3, 8.0, (90.0, 175.0), 500_000, 1),
    "wide9": (9, 7, 2, 40.0, (120.0, 165.0), 900_000, 1),
    "primary16": (16, 16, 4, 15.9, (143.0, 175.0), 1500, 0),
}


def _make(name, dev):
    L = _lib()
    n, na, ns, fwhm, win, J, sc = CASES[name]
    dx = 12.8 / n
    g = synth.Geometry(n, n, dx, n, dx, na, fwhm_e_kev=fwhm, win_lo_kev=win[0], win_hi_kev=win[1], n_subsets=ns,
                       scatter_model=sc)
    X, Y = synth.phantoms.pixel_centres(n, n, dx)
    mu = np.where((X / 5.6) ** 2 + (Y / 5.1) ** 2 <= 1.0, 0.15, 0.0).astype(np.float32)
    act = np.where(X ** 2 + Y ** 2 <= 4.6 ** 2, 1.0, 0.0).astype(np.float32)
    act[np.hypot(X - 1.6, Y + 0.8) < 1.5] = 4.0
    ev = synth.generate_events(g, act, mu, J, 5)
    if name == "odd21":
        keep = ev["angle"] % 6 != 5
        ev = {k: ev[k][keep] for k in ("angle", "u_bin", "energy")}
    return L, g.as_dict(), act, mu, {k: ev[k] for k in ("angle", "u_bin", "energy")}


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_flux_means_and_backprojection_match_oracle(dev, name, masked):
    L, g, act, mu, ev = _make(name, dev)
    m = O.OracleModel(g, mu)
    mask = (act >= 2) if masked else (mu > 0)
    q_em = np.flatnonzero(mask.ravel() & (mu.ravel() > 0)).astype(np.int32)
    ctx = L.Context(g, torch.as_tensor(mu, device=dev),
                    emission=torch.as_tensor(mask.astype(np.float32), device=dev) if masked else None)
    try:
        evd = L.events_to_device(ev, dev)
        J = len(ev["angle"])
        got = ctx.forward(evd, torch.as_tensor(act, device=dev)).cpu().numpy()
        w = synth.random_weights(J, 3)
        back = ctx.backproject(evd, torch.as_tensor(w, device=dev)).cpu().numpy().ravel()
    finally:
        ctx.close()
    idx = np.sort(np.random.default_rng(1).choice(J, 1500, replace=False))
    ref = m.system_matrix({k: ev[k][idx] for k in ev}, q_em) @ act.ravel()[q_em].astype(np.float64)
    live = ref > 1e-12 * ref.max()
    rel = np.abs(got[idx] - ref)[live] / ref[live]
    print(name, masked, "means: max", rel.max(), "rms", np.sqrt(np.mean(rel ** 2)), flush=True)
    assert live.sum() > 500 and rel.max() <= (1e-4 if masked else 2e-5)
    q = np.sort(np.random.default_rng(2).choice(q_em, min(4, len(q_em)), replace=False)).astype(np.int32)
    step = max(1, J // 60_000)   # a share of the events' rows is enough for the oracle's time
    part = np.arange(0, J, step)
    if step > 1:
        ctx = L.Context(g, torch.as_tensor(mu, device=dev),
                        emission=torch.as_tensor(mask.astype(np.float32), device=dev) if masked else None)
        wz = np.zeros_like(w)
        wz[part] = w[part]
        try:
            back = ctx.backproject(evd, torch.as_tensor(wz, device=dev)).cpu().numpy().ravel()
        finally:
            ctx.close()
    bref = m.system_matrix({k: ev[k][part] for k in ev}, q).T @ w[part].astype(np.float64)
    err = np.abs(back[q] - bref) / bref
    print(name, masked, "back:", err.max(), flush=True)
    assert err.max() <= 5e-6
    assert np.all(back[np.setdiff1d(np.arange(mu.size), q_em)] == 0)


@pytest.mark.parametrize("name", ["disk16", "odd21"])
def test_flux_batch_equals_single_runs_and_cached_rows(dev, name):
    """Three realisations (one empty) in a batch, bit for bit each one's own
    run, and against the term-by-term rows that a row cache keeps."""
    L, g, act, mu, ev = _make(name, dev)
    J = len(ev["angle"])
    offs = [0, J, J, J + J]
    cat = L.events_to_device({k: np.concatenate([ev[k], ev[k][::-1]]) for k in ev}, dev)
    one = [L.events_to_device(ev, dev), L.events_to_device({k: ev[k][::-1].copy() for k in ev}, dev)]
    start = (mu > 0).astype(np.float32)
    ctx = L.Context(g, torch.as_tensor(mu, device=dev))
    try:
        batch = ctx.reconstruct(cat, 2, batch_offsets=offs).cpu().numpy()
        for r, e in ((0, one[0]), (2, one[1])):
            assert np.array_equal(batch[r], ctx.reconstruct(e, 2).cpu().numpy()), r
        assert not batch[1].any()
        evs = L.lmosem_events_load(ctx.handle, one[0])
        try:
            L.lmosem_cache_rows(ctx.handle, evs, True)
            img = torch.as_tensor(start, device=dev).contiguous()
            ll = L.lmosem_iterate(ctx.handle, evs, 2, img, want_loglik=True)
            rows = img.cpu().numpy()
            L.lmosem_cache_rows(ctx.handle, evs, False)
            img = torch.as_tensor(start, device=dev).contiguous()
            ll2 = L.lmosem_iterate(ctx.handle, evs, 2, img, want_loglik=True)
            flux = img.cpu().numpy()
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()
    assert np.array_equal(flux, batch[0])
    on = mu > 0
    assert np.max(np.abs(flux - rows)[on] / np.maximum(rows[on], 1e-3 * rows.max())) <= 1e-4
    np.testing.assert_allclose(ll2, ll, rtol=1e-6)


def test_primary_batch_with_fewer_events_than_slots(dev):
    """Four realisations of 10 events on 16 angles, without scatter: the
    workspace (no larger than the rows of the events) takes the slots in more
    than one chunk, so that backprojection and update run apart; bit for bit
    each realisation's own run, where they are one kernel."""
    L, g, act, mu, ev = _make("primary16", dev)
    g = dict(g, n_subsets=1)
    pick = {k: ev[k][:40] for k in ev}
    cat = L.events_to_device(pick, dev)
    ctx = L.Context(g, torch.as_tensor(mu, device=dev))
    try:
        batch = ctx.reconstruct(cat, 2, batch_offsets=[0, 10, 20, 30, 40]).cpu().numpy()
        for r in range(4):
            one = L.events_to_device({k: pick[k][10 * r:10 * r + 10].copy() for k in pick}, dev)
            assert np.array_equal(batch[r], ctx.reconstruct(one, 2).cpu().numpy()), r
    finally:
        ctx.close()
    assert batch.any()


# 560 support pixels, where the path table is filled on demand: few events per
# realisation go term by term (the first two), many through the flux stages
@pytest.mark.parametrize("per_real,n_real", [(60, 1), (150, 5), (200_000, 1)])
def test_iterated_sets_by_size_equal_cached_rows(dev, per_real, n_real):
    L = _lib()
    g = synth.Geometry(32, 32, 0.4, 32, 0.4, 16, n_subsets=2)
    X, Y = synth.phantoms.pixel_centres(32, 32, 0.4)
    mu = np.where((X / 5.6) ** 2 + (Y / 5.1) ** 2 <= 1.0, 0.15, 0.0).astype(np.float32)
    assert (mu > 0).sum() >= 512
    J = per_real * n_real
    ev = synth.generate_events(g, (mu > 0).astype(np.float32), mu, J, 9)
    evd = L.events_to_device({k: ev[k] for k in ("angle", "u_bin", "energy")}, dev)
    offs = list(range(0, J + 1, per_real)) if n_real > 1 else None
    img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).expand(n_real, -1, -1).contiguous().clone()
    rows = img.clone()
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev))
    try:
        evs = L.lmosem_events_load(ctx.handle, evd, offs)
        try:
            L.lmosem_iterate(ctx.handle, evs, 2, img, n_real=n_real)
            L.lmosem_cache_rows(ctx.handle, evs, True)
            L.lmosem_iterate(ctx.handle, evs, 2, rows, n_real=n_real)
        finally:
            L.lmosem_events_free(evs)
        rec = ctx.reconstruct(evd, 2, batch_offsets=offs).reshape(img.shape)
        again = ctx.reconstruct(evd, 2, batch_offsets=offs).reshape(img.shape)
    finally:
        ctx.close()
    on = np.broadcast_to(mu > 0, img.shape)
    a = rows.cpu().numpy().astype(np.float64)[on]
    for b in (img.cpu().numpy()[on], rec.cpu().numpy()[on]):
        assert np.max(np.abs(b - a) / np.maximum(a, 1e-3 * a.max())) <= 1e-4
    assert torch.equal(rec, again)


def test_path_table_in_two_passes(dev):
    """A path table whose direction terms (100x100 px, 120 angles: 95 MB) are
    formed in two runs of angles: two iterations of a small set, which go term
    by term, against the oracle (bar of the term-by-term path, 1e-4)."""
    L = _lib()
    g = synth.Geometry(100, 100, 0.128, 100, 0.128, 120, n_subsets=1)
    X, Y = synth.phantoms.pixel_centres(100, 100, 0.128)
    mu = np.where((X / 1.9) ** 2 + (Y / 1.6) ** 2 <= 1.0, 0.15, 0.0).astype(np.float32)
    assert (mu > 0).sum() >= 512
    ev = synth.generate_events(g, (mu > 0).astype(np.float32), mu, 300, 4)
    ev = {k: ev[k] for k in ("angle", "u_bin", "energy")}
    m = O.OracleModel(g.as_dict(), mu)
    img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).contiguous()
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev))
    try:
        evs = L.lmosem_events_load(ctx.handle, L.events_to_device(ev, dev))
        try:
            L.lmosem_iterate(ctx.handle, evs, 2, img)
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()
    ref, _ = O.os_lm_mlem(m.system_matrix(ev), ev["angle"], m.sensitivity(-1)[None, :], 2, np.ones(len(m.support)), 1)
    got = img.cpu().numpy().ravel()[m.support]
    assert np.max(np.abs(got - ref) / np.maximum(ref, 1e-3 * ref.max())) <= 1e-4
