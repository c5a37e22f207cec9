"""Contexts that are changed while they are members of a batch, and batch members against the same
runs alone."""
from __future__ import annotations

import pytest

import picgen
from tests.test_gpu_batch import TOL64, TOLMIX, compare
from tests.test_gpu_batch import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu

GUARD = 1 << 16   # bytes after every block


@pytest.fixture
def guarded(pic):  # noqa: F811
    """The library's device memory in blocks of exactly the size asked for, followed by a guard;
    yields a function that says which blocks' guards were written."""
    import torch
    blocks = []

    def alloc(nbytes, device):
        t = torch.full((nbytes + GUARD,), 0xA5, dtype=torch.uint8, device=f"cuda:{device}")
        torch.cuda.synchronize()
        blocks.append((nbytes, t))
        return t.data_ptr()

    pic.set_allocator(alloc, lambda ptr, nbytes, device: None)   # (kept to the end)
    try:
        yield lambda: [n for n, t in blocks if not bool((t[n:] == 0xA5).all())]
    finally:
        pic.set_allocator(None, None)


def plasma(nx, nz, ppc, seed, mixed):
    wl = picgen.random_small(seed, nx=nx, nz=nz, ppc=ppc, bc_x=0, dx=0.5, dz=0.4, dt=0.3)
    return picgen.fp32_representable(wl) if mixed else wl


def load(ctx, wl):
    for s, sp in enumerate(wl.species):
        ctx.load_particles(s, sp.q, sp.m, sp.w, sp.xi_x, sp.xi_z, sp.ux, sp.uy, sp.uz)


@pytest.mark.parametrize("mixed", [0, 1])
@pytest.mark.parametrize("nx,nz,before,after,tiles", [
    (64, 64, 4, 64, None), (64, 64, 4, 16, None), (192, 96, 1, 128, None), (64, 64, 16, None, (64, 1))])
def test_member_reloaded_then_alone(pic, guarded, nx, nz, before, after, tiles, mixed):  # noqa: F811
    """Reloaded with another number of particles per cell, or given a fixed tile shape and then the
    automatic one, inside the batch; then alone again: no write past any array, and the results of
    the run that never was a member."""
    print(f"[gpu-case] member {nx}x{nz} {before} -> {after} tiles {tiles} mixed {mixed}", flush=True)
    wl = plasma(nx, nz, before, 5, mixed)
    ctx, solo = (pic.Context(wl.grid, precision=mixed, track_ids=True, tile=tiles or (0, 0)) for _ in range(2))
    for c in (ctx, solo):
        load(c, wl)
    batch = pic.Batch(0, mixed)
    batch.add(ctx)
    batch.step(1)
    solo.step(1)
    for c in (ctx, solo):
        if after:
            load(c, plasma(nx, nz, after, 6, mixed))
        if tiles:
            c.set_tiles(0, 0)
    batch.step(2)
    solo.step(2)
    batch.remove(ctx)
    for c in (ctx, solo):
        c.step(2)
    compare(ctx, solo, len(wl.species), TOLMIX if mixed else TOL64)
    assert guarded() == []
    for x in (batch, ctx, solo):
        x.close()
