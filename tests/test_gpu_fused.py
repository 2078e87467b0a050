"""Sub-iterations term by term in one kernel (emission sets that one workgroup
covers) against the FP64 oracle: from one wave of pixels to the widest set that
runs this way and the first that does not, tiles of 8, 16 and 32 events with
remainders, three realisations (one empty) and angles without events.

Tolerance: the term-by-term path's bar of 1e-4 a mean carried through three
iterations' sums, relative to each pixel above a thousandth of the maximum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle as O  # noqa: E402
import synth  # noqa: E402


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("n", [9, 16, 20, 26, 28])   # 45, 140, 220, 372 and 428 pixels
def test_iterations_match_oracle(n, tile):
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    dx = 12.8 / n
    g = synth.Geometry(n, n, dx, n, dx, 12, n_subsets=2)
    X, Y = synth.phantoms.pixel_centres(n, n, dx)
    mu = np.where((X / 5.6) ** 2 + (Y / 5.1) ** 2 <= 1.0, 0.15, 0.0).astype(np.float32)
    ev = synth.generate_events(g, (mu > 0).astype(np.float32), mu, 700, 3)
    ev = {k: ev[k] for k in ("angle", "u_bin", "energy")}
    keep = (ev["angle"] != 4) | (np.arange(700) < 300)   # the last realisation misses an angle
    ev = {k: v[keep] for k, v in ev.items()}
    J = int(keep.sum())
    offs = [0, 300, 300, J]
    m = O.OracleModel(g.as_dict(), mu)
    sens = np.stack([m.sensitivity(i) for i in range(2)])
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev))
    try:
        L.lmosem_set_tuning(ctx.handle, tile)
        evs = L.lmosem_events_load(ctx.handle, L.events_to_device(ev, dev), offs)
        try:
            img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).expand(3, -1, -1).contiguous().clone()
            ll = L.lmosem_iterate(ctx.handle, evs, 3, img, n_real=3, want_loglik=True)
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()
    got = img.cpu().numpy().reshape(3, -1)[:, m.support]
    assert not got[1].any()
    for r in (0, 2):
        e = {k: v[offs[r]:offs[r + 1]] for k, v in ev.items()}
        ref, ll_ref = O.os_lm_mlem(m.system_matrix(e), e["angle"], sens, 3, np.ones(len(m.support)), 2)
        err = np.abs(got[r] - ref) / np.maximum(ref, 1e-3 * ref.max())
        assert err.max() <= 1e-4, (r, err.max())
        np.testing.assert_allclose(ll[r], ll_ref, rtol=1e-5)


def test_stored_plans_of_both_forms(tmp_path, monkeypatch):
    """A stored plan names its form by its key: with and without " fused" the
    autotuner takes the line as it stands, and both forms' iterations agree."""
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    w = synth.workload("tiny")
    act, mu = synth.phantom(w)
    evd = L.events_to_device(synth.workload_events(w, n_events=1500), dev)
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LMOSEM_TUNE_CACHE", str(cache))
    ctx = L.Context(w.geom.as_dict(), torch.as_tensor(mu, device=dev))
    out = {}
    try:
        for suffix in (None, "", " fused"):
            if suffix is not None:
                cache.write_text(f"{key}{suffix}|16 512 0 1\n")
            evs = L.lmosem_events_load(ctx.handle, evd)
            try:
                plan = L.lmosem_autotune(ctx.handle, evs)
                if suffix is None:
                    key = cache.read_text().splitlines()[-1].split("|")[0].removesuffix(" fused")
                else:
                    assert plan == (16, 512, 0)
                img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).contiguous()
                L.lmosem_iterate(ctx.handle, evs, 3, img)
                out[suffix] = img.cpu().numpy()
            finally:
                L.lmosem_events_free(evs)
    finally:
        ctx.close()
    on = mu > 0
    for a in (out[""], out[" fused"]):
        assert np.max(np.abs(a - out[None])[on] / np.maximum(out[None][on], 1e-3 * out[None].max())) <= 1e-4
