"""Batches whose subsets have unequal angle lists (17 angles in 3 subsets: 6, 6
and 5), through directional flux, against the rows that a row cache keeps.

A batch's workspace is bounded by the events of its largest subset, so that
small batches take their realisations in groups.  Where the long lists leave
room for fewer realisations at a time than the short one, the estimate that a
sub-iteration leaves in the workspace must still be the one that the next one
reads.  The sizes in between are some 80 rows wide; the event counts below step
through them by less, over one to all realisations a group.

Tolerance: means agree within 2e-5 (a path's interpolation error in the far
tails; the bulk within 2e-7), and an estimate after two iterations of three
subsets carries six of them: 1.2e-4 at most, 1e-4 held."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import synth  # noqa: E402


@pytest.mark.parametrize("n_real", [2, 3])
def test_unequal_subset_lists_match_cached_rows(n_real):
    from paper_2002_12471_amd import lmosem as L
    dev = torch.device("cuda:0")
    n = 48
    dx = 12.8 / n
    g = synth.Geometry(n, n, dx, n, dx, 17, fwhm_u_cm=2.0, n_subsets=3)
    X, Y = synth.phantoms.pixel_centres(n, n, dx)
    mu = np.where((X / 5.6) ** 2 + (Y / 5.1) ** 2 <= 1.0, 0.15, 0.0).astype(np.float32)
    on = np.broadcast_to(mu > 0, (n_real, n, n))
    rng = np.random.default_rng(7)
    start = np.where(on, rng.uniform(0.5, 4.0, (n_real, n, n)), 0.0).astype(np.float32)   # each realisation its own
    total = 16_000
    ev = synth.generate_events(g, (mu > 0).astype(np.float32), mu, total, 5)
    ev = {k: ev[k] for k in ("angle", "u_bin", "energy")}
    ctx = L.Context(g.as_dict(), torch.as_tensor(mu, device=dev))
    tried = 0
    try:
        # a largest subset has 6/17 of the events
        for rows in range(700 * n_real, 1700 * n_real, 36):
            J = rows * 17 // 6
            if J > total:
                break
            offs = [J * r // n_real for r in range(n_real + 1)]
            evs = L.lmosem_events_load(ctx.handle, L.events_to_device({k: ev[k][:J] for k in ev}, dev), offs)
            try:
                got = torch.as_tensor(start, device=dev).contiguous().clone()
                L.lmosem_set_timing(ctx.handle, True)
                before = ctx.stats()["forward_launches"]
                L.lmosem_iterate(ctx.handle, evs, 2, got, n_real=n_real)
                torch.cuda.synchronize()
                stages = ctx.stats()["forward_launches"] - before
                L.lmosem_set_timing(ctx.handle, False)
                if stages < 2 * 6:   # (one forward launch a sub-iteration: term by term)
                    continue
                tried += 1
                L.lmosem_cache_rows(ctx.handle, evs, True)
                rows_img = torch.as_tensor(start, device=dev).contiguous().clone()
                L.lmosem_iterate(ctx.handle, evs, 2, rows_img, n_real=n_real)
            finally:
                L.lmosem_events_free(evs)
            a, b = rows_img.cpu().numpy().astype(np.float64), got.cpu().numpy()
            for r in range(n_real):
                x, y = a[r][on[r]], b[r][on[r]]
                err = np.max(np.abs(y - x) / np.maximum(x, 1e-3 * x.max()))
                assert err <= 1e-4, (J, r, stages, err)
    finally:
        ctx.close()
    assert tried >= 25
