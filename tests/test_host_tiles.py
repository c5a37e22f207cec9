"""Tile bookkeeping of contexts that join, change and leave a batch, on the CPU.

The library's host files are compiled against stand-ins for the HIP calls (fake_hip.cpp): memory
has exactly the size asked for, and every launch checks the tile arrays its kernel would write.
The kernels themselves do not run.
"""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import pytest

import picgen
from paper_1308_2590_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1308_2590_amd", "csrc")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "libfake.so")
    # (symbolic: the stand-ins, not a HIP runtime that torch has loaded)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, "-o", lib, os.path.join(ROOT, "tests", "fake_hip.cpp"),
                           os.path.join(CSRC, "pic_capi.cpp"), os.path.join(CSRC, "pic_batch.cpp")])
    saved, binding._lib = binding._lib, None
    try:
        yield binding.load_library(lib)
    finally:
        binding._lib = saved


def load(ctx, wl):
    for s, sp in enumerate(wl.species):
        ctx.load_particles(s, sp.q, sp.m, sp.w, sp.xi_x, sp.xi_z, sp.ux, sp.uy, sp.uz)


def plasma(nx, nz, ppc):
    return picgen.random_small(5, nx=nx, nz=nz, ppc=ppc, bc_x=0, dx=0.5, dz=0.4, dt=0.3)


@pytest.mark.parametrize("mixed", [0, 1])
@pytest.mark.parametrize("leave", ["remove", "destroy"])
@pytest.mark.parametrize("nx,nz,before,after,tiles", [
    (64, 64, 4, 64, None), (64, 64, 4, 16, None), (192, 96, 1, 128, None), (37, 29, 3, 40, None),
    (64, 64, 64, 4, None), (64, 64, 16, None, (64, 1)), (64, 64, 16, None, (1, 1))])
def test_tile_arrays_hold_the_tiles_of_a_member_that_leaves(fake, nx, nz, before, after, tiles, leave, mixed):
    """A member is reloaded with another number of particles per cell, or given a fixed tile shape
    and then the automatic one, inside the batch; then it leaves and is stepped alone."""
    short = fake.fake_short_arrays()
    wl = plasma(nx, nz, before)
    ctx = binding.Context(wl.grid, precision=mixed, tile=tiles or (0, 0))
    load(ctx, wl)
    batch = binding.Batch(0, mixed)
    batch.add(ctx)
    batch.step(1)
    if after:
        load(ctx, plasma(nx, nz, after))
    if tiles:
        ctx.set_tiles(0, 0)
    batch.step(2)
    batch.close() if leave == "destroy" else batch.remove(ctx)
    ctx.step(2)
    assert fake.fake_short_arrays() == short
    ctx.close()
    if leave == "remove":
        batch.close()


def test_member_takes_no_tile_shape_that_it_cannot_keep_alone(fake):
    """22 x 24 cells fit the LDS (163,840 bytes) in the grouped form (here 160,224 bytes) but not in
    the form of a mixed run alone (164,992): refused in the batch as it is outside, and the old
    shape stays."""
    wl = plasma(64, 64, 16)
    ctx, other = binding.Context(wl.grid, precision=1), binding.Context(wl.grid, precision=1)
    load(ctx, wl)
    load(other, wl)
    batch = binding.Batch(0, 1)
    batch.add(ctx)
    for c in (ctx, other):
        old = c.get_info()["tile"]
        with pytest.raises(binding.PicError) as e:
            c.set_tiles(22, 24)
        assert e.value.status == 1 and c.get_info()["tile"] == old
    batch.step(1)
    batch.remove(ctx)
    ctx.step(1)
    for x in (batch, ctx, other):
        x.close()


def test_batch_does_not_step_freed_arrays_after_a_refused_load(fake):
    """Densities per particle take another KB of LDS, which 20 x 26 cells do not leave: the load
    fails after the species' old arrays are gone."""
    wl = plasma(64, 64, 4)
    ctx, other = binding.Context(wl.grid, precision=1, tile=(20, 26)), binding.Context(wl.grid, precision=1)
    load(ctx, wl)
    load(other, wl)
    batch = binding.Batch(0, 1)
    batch.add(ctx)
    batch.add(other)
    batch.step(1)
    short = fake.fake_short_arrays()
    with pytest.raises(binding.PicError) as e:
        load(ctx, picgen.with_particle_densities(plasma(64, 64, 64), seed=3))
    assert e.value.status == 1
    try:
        batch.step(1)   # (may refuse the member's shape)
    except binding.PicError:
        pass
    assert fake.fake_short_arrays() == short
    for x in (batch, ctx, other):
        x.close()


@pytest.fixture
def short_of_memory(fake):
    """The library's memory through a hook that returns none while the yielded list is not empty."""
    refuse = []
    fake.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    fake.hipFree.argtypes = [C.c_void_p]

    def alloc(nbytes, device):
        p = C.c_void_p()
        return 0 if refuse or fake.hipMalloc(C.byref(p), nbytes) else p.value

    binding.set_allocator(alloc, lambda ptr, nbytes, device: fake.hipFree(ptr))
    try:
        yield refuse
    finally:
        binding.set_allocator(None, None)


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("how", ["tiles", "fields"])
def test_without_memory_for_more_tiles_the_old_ones_stay(fake, short_of_memory, how, batched):
    wl = plasma(64, 64, 16)
    ctx = binding.Context(wl.grid, tile=(16, 16))
    load(ctx, wl)
    batch = binding.Batch(0, 0)
    if batched:
        batch.add(ctx)
        batch.step(1)
    short = fake.fake_short_arrays()
    short_of_memory.append(True)
    with pytest.raises(binding.PicError) as e:
        ctx.set_tiles(1, 1)
    assert e.value.status == 2 and ctx.get_info()["tile"] == (16, 16)
    if how == "fields":
        ctx.load_fields(None, None)
    (batch if batched else ctx).step(2)
    assert fake.fake_short_arrays() == short
    del short_of_memory[:]
    ctx.set_tiles(1, 1)
    (batch if batched else ctx).step(1)
    assert fake.fake_short_arrays() == short
    batch.close()
    ctx.close()


@pytest.mark.parametrize("how", ["memory", "too large"])
def test_a_refused_shape_leaves_the_one_that_the_tile_list_is_for(fake, short_of_memory, how):
    """The library's choice follows the particles, which have moved since the load (here none is
    left after a cycle, as the kernels do not run): a refused call must not make it again."""
    wl = picgen.with_particle_densities(plasma(256, 64, 16), seed=3)
    ctx = binding.Context(wl.grid, precision=1 if how == "too large" else 0)
    load(ctx, wl)
    before = ctx.get_info()["tile"]
    ctx.step(1)
    if how == "memory":
        short_of_memory.append(True)
    with pytest.raises(binding.PicError) as e:
        ctx.set_tiles(*((1, 1) if how == "memory" else (64, 64)))
    assert e.value.status == (2 if how == "memory" else 1)
    assert ctx.get_info()["tile"] == before
    ctx.step(1)
    ctx.close()


@pytest.mark.parametrize("then", ["step", "add", "batched"])
def test_a_load_without_memory_for_its_tiles_is_not_stepped(fake, then):
    """16 x 4 cells, which a batch member takes at 12 per cell, need more than the tile arrays hold;
    the shape that the context takes alone fits them, but they list the last load's tiles."""
    refuse = []
    fake.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    fake.hipFree.argtypes = [C.c_void_p]

    def alloc(nbytes, device):
        p = C.c_void_p()
        return 0 if nbytes in refuse or fake.hipMalloc(C.byref(p), nbytes) else p.value

    binding.set_allocator(alloc, lambda ptr, nbytes, device: fake.hipFree(ptr))
    try:
        ctx = binding.Context(plasma(256, 256, 2).grid)
        load(ctx, plasma(256, 256, 2))
        assert ctx.get_info()["tile"] == (32, 4)   # 512 tiles
        batch = binding.Batch(0, 0)
        if then == "batched":
            batch.add(ctx)
        refuse += [1024, 4 * 1025]
        with pytest.raises(binding.PicError) as e:
            load(ctx, plasma(256, 256, 12))
        assert e.value.status == 2
        with pytest.raises(binding.PicError) as e:
            batch.add(ctx) if then == "add" else batch.step(1) if then == "batched" else ctx.step(1)
        assert e.value.status == 4
        alone = ctx.get_info()["tile"]
        assert (alone == (16, 4)) == (then == "batched")
        del refuse[:]
        ctx.load_fields(None, None)   # (deposits again, and lists the tiles)
        assert ctx.get_info()["tile"] == alone
        (batch if then == "batched" else ctx).step(2)
        batch.close()
        ctx.step(1)
        ctx.close()
    finally:
        binding.set_allocator(None, None)
