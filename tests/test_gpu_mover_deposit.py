"""The two deposits of the mover-option kernel against the oracle at 1e-10: shuffles for few
particles per cell on many cells, matrix cores with accumulators for a block's first 24 cells.

Counts per cell on both sides of the line between them (5.5) and of the one where a block's 256
particles fill 24 cells (10.7), grids on both sides of 8192 cells, cells without particles, hot
plasmas, densities per particle.
"""
from __future__ import annotations

import pytest

import picgen
from tests.test_gpu_grouped import thin
from tests.test_gpu_mover import _setup
from tests.test_gpu_parity import check_fields, check_moments, check_particles
from tests.test_gpu_parity import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,nz,ppc,te,keep,dens", [
    (97, 89, 1, 1.0, 1, False), (97, 89, 2, 200.0, 1, True), (131, 127, 5, 1.0, 2, False),
    (97, 89, 5, 200.0, 1, False), (97, 89, 6, 1.0, 1, True), (64, 127, 5, 1.0, 1, False),
    (37, 11, 3, 5.0, 1, False), (37, 11, 9, 200.0, 1, False), (37, 11, 10, 1.0, 3, True),
    (37, 11, 11, 1.0, 1, False), (1, 40, 7, 1.0, 1, False)])
def test_mover_deposits(pic, nx, nz, ppc, te, keep, dens, bc):  # noqa: F811
    bc = bc if nx > 1 else 0
    wl = picgen.random_small(170 + ppc, nx=nx, nz=nz, ppc=ppc, bc_x=bc, dx=0.5, dz=0.4, dt=0.4, temps=(te, 0.5))
    if keep > 1:
        thin(wl, keep)
    if dens:
        wl = picgen.with_particle_densities(wl, seed=ppc)
    print(f"[gpu-case] mover deposit {nx}x{nz} ppc={ppc} te={te} keep={keep} densities={dens} bc={bc}", flush=True)
    ctx, orc = _setup(pic, wl, 3, ppc)
    check_moments(ctx, orc)
    ctx.step(2)
    orc.step(2)
    check_fields(ctx, orc)
    check_moments(ctx, orc)
    check_particles(ctx, orc, wl)
    assert ctx.get_info()["overflow_flags"] == 0
    ctx.close()
