"""The memory cap where sets run through directional flux: what a row cache
brings with it is asked for before it is allocated, and counted."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import synth  # noqa: E402


def _lib():
    from paper_2002_12471_amd import lmosem as L
    return L


def _context(n_subsets):
    L, dev = _lib(), torch.device("cuda:0")
    w = synth.workload("brain64")
    _, mu = synth.phantom(w)
    g = dict(w.geom.as_dict(), n_subsets=n_subsets)
    return L, dev, L.Context(g, torch.as_tensor(mu, device=dev)), w, mu


def _stages(L, ctx, evs, img, n_iters=1):
    """forward launches of n_iters iterations with timing on"""
    L.lmosem_set_timing(ctx.handle, True)
    before = ctx.stats()["forward_launches"]
    L.lmosem_iterate(ctx.handle, evs, n_iters, img)
    torch.cuda.synchronize()
    n = ctx.stats()["forward_launches"] - before
    L.lmosem_set_timing(ctx.handle, False)
    return n


def test_row_cache_asks_for_its_rows_too():
    """One subset: the rows that the cache's kernels work with are as large as
    the cache.  A cap with room for the cache alone refuses it."""
    L, dev, ctx, w, mu = _context(1)
    J = 40_000
    ev = L.events_to_device(synth.workload_events(w, n_events=J), dev)
    cache = 4 * J * 1472
    try:
        evs = L.lmosem_events_load(ctx.handle, ev)
        try:
            img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).contiguous()
            assert _stages(L, ctx, evs, img.clone()) >= 2
            held = L.lmosem_memory_held(ctx.handle)
            L.lmosem_set_memory_cap(ctx.handle, held + cache + (50 << 20))
            with pytest.raises(L.LmosemError) as ei:
                L.lmosem_cache_rows(ctx.handle, evs, True)
            assert ei.value.status == L.ENOMEM
            assert L.lmosem_memory_held(ctx.handle) == held
            L.lmosem_iterate(ctx.handle, evs, 1, img.clone())
            L.lmosem_set_memory_cap(ctx.handle, held + 2 * cache + (50 << 20))
            L.lmosem_cache_rows(ctx.handle, evs, True)
            assert held + 2 * cache <= L.lmosem_memory_held(ctx.handle) <= held + 2 * cache + (50 << 20)
            assert _stages(L, ctx, evs, img.clone()) == 1
            L.lmosem_cache_rows(ctx.handle, evs, False)
            assert held + cache <= L.lmosem_memory_held(ctx.handle) < held + 2 * cache
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()
