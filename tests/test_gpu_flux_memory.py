"""The memory cap where sets run through directional flux: what a row cache
brings with it is asked for before it is allocated, and counted; a cap with room
for the path table and a set term by term admits the set, whatever the flux
tables take; and the stages give way to a set or a row cache that fits only
without them.  Images on either route agree within 1e-4 (the bar of a mean, two
sub-iterations of one subset)."""
import re

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
            L.lmosem_set_memory_cap(ctx.handle, held + 2 * cache + (100 << 20))   # (and the flux tables beside a filled path table)
            L.lmosem_cache_rows(ctx.handle, evs, True)
            assert held + 2 * cache <= L.lmosem_memory_held(ctx.handle) <= held + 2 * cache + (100 << 20)
            assert _stages(L, ctx, evs, img.clone()) == 1
            L.lmosem_cache_rows(ctx.handle, evs, False)
            assert held + cache <= L.lmosem_memory_held(ctx.handle) < held + 2 * cache
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()


def _table_bytes(L, ctx):
    """what the context holds with its path table, by the refusal under a small cap"""
    L.lmosem_set_memory_cap(ctx.handle, 1 << 30)
    with pytest.raises(L.LmosemError) as ei:
        ctx.sensitivity(-1)
    L.lmosem_set_memory_cap(ctx.handle, 0)
    return int(re.search(r"to (\d+) device bytes", str(ei.value)).group(1))


@pytest.mark.parametrize("capped_from_the_start", [False, True])
def test_cap_that_holds_table_and_set_admits_the_set(capped_from_the_start):
    """20,000 events in 8 subsets take some 16 MB term by term."""
    L, dev, ctx, w, mu = _context(8)
    ev = L.events_to_device(synth.workload_events(w, n_events=20_000), dev)
    try:
        cap = _table_bytes(L, ctx) + (18 << 20)
        if not capped_from_the_start:
            ctx.sensitivity(-1)
        L.lmosem_set_memory_cap(ctx.handle, cap)
        evs = L.lmosem_events_load(ctx.handle, ev)
        try:
            assert L.lmosem_memory_held(ctx.handle) <= cap
            img = torch.as_tensor((mu > 0).astype(np.float32), device=dev).contiguous()
            L.lmosem_iterate(ctx.handle, evs, 1, img)
            torch.cuda.synchronize()
            assert bool((img > 0).any())
        finally:
            L.lmosem_events_free(evs)
    finally:
        ctx.close()


def test_stages_give_way_to_a_row_cache():
    """Two sets through the stages; the cap has room for one's row cache only
    without their tables.  Both then run term by term, the second one's images
    as before within the bar."""
    L, dev, ctx, w, mu = _context(8)
    J = 60_000
    cat = synth.workload_events(w, n_events=2 * J)
    parts = [L.events_to_device({k: v[i::2].copy() for k, v in cat.items() if k in ("angle", "u_bin", "energy")}, dev)
             for i in range(2)]
    # beside the cache: some 110 MB with the stages (one set's rows, and the flux
    # tables beside a filled path table), 50 MB without (two sets' rows for their
    # stages' workspaces)
    cache, more = 4 * J * 1472, 82 << 20
    start = torch.as_tensor((mu > 0).astype(np.float32), device=dev).contiguous()
    try:
        ctx.sensitivity(-1)
        sets = [L.lmosem_events_load(ctx.handle, p) for p in parts]
        try:
            before = start.clone()
            assert _stages(L, ctx, sets[1], before) >= 16
            held = L.lmosem_memory_held(ctx.handle)
            cap = held + cache + more
            L.lmosem_set_memory_cap(ctx.handle, cap)
            L.lmosem_cache_rows(ctx.handle, sets[0], True)
            assert held < L.lmosem_memory_held(ctx.handle) <= cap
            first, cached, after = start.clone(), start.clone(), start.clone()
            assert _stages(L, ctx, sets[0], first) == 8 and _stages(L, ctx, sets[0], cached) == 8
            assert _stages(L, ctx, sets[1], after) == 8
            # calls on events of one sub-iteration still work
            L.lmosem_set_memory_cap(ctx.handle, 0)
            m = ctx.forward({k: v[:500].contiguous() for k, v in parts[0].items()}, start)
            assert bool(torch.isfinite(m).all())
        finally:
            for s in sets:
                L.lmosem_events_free(s)
    finally:
        ctx.close()
    x, y = before.double(), after.double()
    on = torch.as_tensor(mu > 0, device=dev)
    assert float(((y - x).abs() / torch.clamp(x, min=1e-3 * float(x.max())))[on].max()) <= 1e-4
    assert torch.allclose(first, cached, rtol=1e-5)
