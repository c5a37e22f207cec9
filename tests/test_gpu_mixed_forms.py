"""Mixed runs in each form, alone and as batch members, against the oracle at the bounds of
test_gpu_mixed: counts per cell around multiples of 16 and 64, cells without particles in between,
tiles of one cell to the widest, plasmas in which a third of the particles change cell.  The load
deposit, then one cycle from identical state."""
from __future__ import annotations

import pytest

import picgen
from tests.pic_checks import abs_deposit_scale
from tests.test_gpu_grouped import thin
from tests.test_gpu_mixed import (check_moments_vs, compare_step, compare_step_unlabelled, setup_both,
                                  species_tuples)
from tests.test_gpu_mixed import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("labels", [True, False])
@pytest.mark.parametrize("tile", [(0, 0), (1, 1), (5, 3), (64, 1)])
@pytest.mark.parametrize("ppc,te,keep,nx", [(1, 5.0, 1, 37), (15, 5.0, 3, 37), (16, 200.0, 1, 37), (17, 200.0, 2, 37),
                                            (64, 5.0, 1, 37), (65, 200.0, 4, 37), (17, 5.0, 1, 2), (65, 200.0, 1, 1)])
def test_mixed_forms(pic, ppc, te, keep, nx, tile, labels, batch):  # noqa: F811
    wl = picgen.random_small(270 + ppc, nx=nx, nz=11, ppc=ppc, bc_x=ppc % 2 if nx > 2 else 0, dx=0.5, dz=0.4, dt=0.4,
                             temps=(te, 0.5))
    if keep > 1:
        thin(wl, keep)
    wl = picgen.fp32_representable(wl)
    print(f"[gpu-case] mixed form nx={nx} ppc={ppc} te={te} keep={keep} tile={tile} labels={labels} batch={batch}",
          flush=True)
    ctx, orc = setup_both(pic, wl, fields=picgen.random_fields(ppc, wl.grid), tile=tile, track_ids=labels)
    parts = [orc.particles(s) for s in range(len(wl.species))]
    scale = abs_deposit_scale(nx, 11, wl.grid.bc_x, wl.grid.dt, species_tuples(wl, parts), orc.H)
    check_moments_vs(ctx.read_moments(), orc.moments(), scale, what="load")
    b = None
    if batch:
        b = pic.Batch(0, 1)
        b.add(ctx)
    prev = [ctx.read_particles(s, ids=True)["id"] for s in range(len(wl.species))] if labels else None
    (b or ctx).step(1)
    orc.step(1)
    if labels:
        compare_step(ctx, orc, wl, prev)
    else:
        compare_step_unlabelled(ctx, orc, wl)
    assert ctx.get_info()["overflow_flags"] == 0
    if b:
        b.close()
    ctx.close()
