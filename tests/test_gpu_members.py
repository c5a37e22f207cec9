"""Contexts that are changed while they are members of a batch, and batch members against the same
runs alone."""
from __future__ import annotations

import pytest

import picgen
from tests.test_gpu_batch import TOL64, TOLMIX, compare, rel
from tests.test_gpu_batch import pic  # noqa: F401  -- fixture
from tests.test_gpu_parity import check_fields, check_moments, check_particles, setup_both

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


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("labels", [True, False])
def test_mixed_member_and_the_run_alone(pic, labels, graph):  # noqa: F811
    """A mixed member adds its particles' FP32 moments in FP64.  Alone, a run in the direct form by
    its tiles does the same: only the order of the additions differs (TOL64).  A run of lane sums, or
    direct for its few particles per lane, rounds to 32 bits on the way: moments within TOLMIX.  With
    densities per particle in some, which must not change the others, and joining at other cycles."""
    shapes = [(64, 48, 40, 0), (37, 29, 20, 1), (9, 7, 100, 1), (39, 1037, 3, 0), (20, 17, 2, 1), (16, 1026, 9, 1)]
    wls = [plasma(nx, nz, ppc, 40 + i, 0) for i, (nx, nz, ppc, _) in enumerate(shapes)]
    wls = [picgen.fp32_representable(picgen.with_particle_densities(wl, seed=3) if s[3] else wl)
           for wl, s in zip(wls, shapes)]
    print(f"[gpu-case] mixed members and runs alone, labels {labels} graph {graph}", flush=True)
    mem, solo = ([pic.Context(wl.grid, precision=1, track_ids=labels) for wl in wls] for _ in range(2))
    for cs in (mem, solo):
        for c, wl in zip(cs, wls):
            load(c, wl)
    batch = pic.Batch(0, 1)
    batch.set_graph(graph)
    for c in mem[::2]:
        batch.add(c)
    batch.step(1)
    for c in mem[1::2]:
        c.step(1)
        batch.add(c)
    batch.step(2)
    batch.remove(mem[0])
    mem[0].step(1)
    batch.step(1)
    for c, s, wl, (nx, nz, ppc, _) in zip(mem, solo, wls, shapes):
        s.step(4)
        same(c, s, len(wl.species), labels, TOL64 if nz > 1000 else TOLMIX)
    for x in (batch, *mem, *solo):
        x.close()


def same(a, b, nsp, labels, tol):
    ma, mb = a.read_moments(), b.read_moments()
    for p in range(ma.shape[0]):
        assert rel(ma[p], mb[p]) <= tol, f"moment plane {p}: {rel(ma[p], mb[p]):.2e}"
    for x, y in zip(a.read_fields(), b.read_fields()):
        assert rel(x, y) <= tol
    for s in range(nsp):
        pa, pb = a.read_particles(s, ids=labels), b.read_particles(s, ids=labels)
        for k in pa:
            assert rel(pa[k], pb[k]) <= tol, f"species {s} {k}"


@pytest.mark.parametrize("labels", [True, False])
def test_member_forms_in_64_bits(pic, labels):  # noqa: F811
    """Members in the direct form and in the grouped one with each of the batch's tile widths, beside
    each other, against the oracle at 1e-10."""
    shapes = [(39, 1037, 3, 0), (16, 1026, 9, 1), (130, 33, 2, 0), (130, 33, 7, 1), (96, 21, 6, 0), (95, 21, 6, 1),
              (64, 9, 17, 0), (63, 9, 30, 0), (5, 4, 65, 1)]
    print(f"[gpu-case] member forms in 64 bits, labels {labels}", flush=True)
    batch = pic.Batch(0, 0)
    runs = []
    for i, (nx, nz, ppc, bc) in enumerate(shapes):
        wl = picgen.random_small(60 + i, nx=nx, nz=nz, ppc=ppc, bc_x=bc, dx=0.5, dz=0.4, dt=0.4, temps=(50.0, 0.5))
        runs.append((wl, *setup_both(pic, wl, fields=picgen.random_fields(i, wl.grid), track_ids=labels)))
        batch.add(runs[-1][1])
    batch.step(2)
    for wl, ctx, orc in runs:
        orc.step(2)
        check_fields(ctx, orc)
        check_moments(ctx, orc)
        check_particles(ctx, orc, wl, ids=labels)
        assert ctx.get_info()["overflow_flags"] == 0
    for _, ctx, _ in runs:
        batch.remove(ctx)
        ctx.close()
    batch.close()
