"""The particle kernel's direct form with labels and with densities per particle, alone and as a
member of a batch, against the oracle: 64 bits at 1e-10, mixed at the bounds of test_gpu_mixed."""
from __future__ import annotations

import pytest

import picgen
from tests import test_gpu_mixed, test_gpu_parity
from tests.test_gpu_parity import check_fields, check_moments, check_particles
from tests.test_gpu_parity import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("labels", [False, True])
@pytest.mark.parametrize("mixed", [0, 1])
@pytest.mark.parametrize("nx,nz,ppc,te,bc,dens,tile", [
    (39, 1037, 3, 200.0, 0, True, (0, 0)), (16, 1026, 9, 1.0, 1, True, (0, 0)), (39, 1037, 1, 5.0, 1, False, (0, 0)),
    (37, 11, 2, 5.0, 0, True, (5, 3)), (20, 17, 4, 200.0, 1, True, (1, 1)), (65, 9, 3, 5.0, 0, False, (64, 1)),
    (1, 8, 6, 5.0, 0, True, (0, 0))])
def test_direct_form(pic, nx, nz, ppc, te, bc, dens, tile, mixed, labels, batch):  # noqa: F811
    wl = picgen.random_small(190 + ppc, nx=nx, nz=nz, ppc=ppc, bc_x=bc, dx=0.5, dz=0.4, dt=0.4, temps=(te, 0.5))
    if dens:
        wl = picgen.with_particle_densities(wl, seed=ppc)
    if mixed:
        wl = picgen.fp32_representable(wl)
    print(f"[gpu-case] direct {nx}x{nz} ppc={ppc} te={te} bc={bc} densities={dens} tile={tile} mixed={mixed} "
          f"labels={labels} batch={batch}", flush=True)
    side = test_gpu_mixed if mixed else test_gpu_parity
    ctx, orc = side.setup_both(pic, wl, fields=picgen.random_fields(3, wl.grid), tile=tile, track_ids=labels)
    b = None
    if batch:
        b = pic.Batch(0, mixed)
        b.add(ctx)
    prev = [ctx.read_particles(s, ids=True)["id"] for s in range(len(wl.species))] if labels else None
    cycles = 1 if mixed else 2
    (b or ctx).step(cycles)
    orc.step(cycles)
    if not mixed:
        check_fields(ctx, orc)
        check_moments(ctx, orc)
        check_particles(ctx, orc, wl, ids=labels)
    elif labels:
        test_gpu_mixed.compare_step(ctx, orc, wl, prev)
    else:
        test_gpu_mixed.compare_step_unlabelled(ctx, orc, wl)
    assert ctx.get_info()["overflow_flags"] == 0
    if b:
        b.close()
    ctx.close()
