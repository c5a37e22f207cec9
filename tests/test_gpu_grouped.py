"""The particle kernel's two forms where they can go wrong, against the oracle at 1e-10.

The grouped form takes 64 slots per wavefront and sums them per cell through the matrix cores, 16
lanes at a time: particle counts around multiples of 16 and 64 per cell, cells without particles
in between, tiles of one cell to the widest, and hot plasmas in which a third of the particles
change cell every cycle.  The direct form is chosen at few particles per cell on grids of many
tiles.  Runs without labels use their own kernel instantiations, so both are run.
"""
from __future__ import annotations

import numpy as np
import pytest

import picgen
from tests.test_gpu_parity import check_fields, check_moments, check_particles, setup_both
from tests.test_gpu_parity import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


def thin(wl, keep):
    """Only every keep-th cell column occupied."""
    for sp in wl.species:
        on = np.floor(sp.xi_x).astype(int) % keep == 0
        for k in ("xi_x", "xi_z", "ux", "uy", "uz"):
            setattr(sp, k, np.ascontiguousarray(getattr(sp, k)[on]))
    return wl


@pytest.mark.parametrize("ids", [True, False])
@pytest.mark.parametrize("tile", [(0, 0), (1, 1), (5, 3), (8, 4), (64, 1)])
@pytest.mark.parametrize("ppc,te,keep", [(1, 5.0, 1), (15, 5.0, 3), (16, 200.0, 1), (17, 200.0, 2),
                                         (64, 5.0, 1), (65, 200.0, 4)])
def test_grouped_form(pic, ppc, te, keep, tile, ids):  # noqa: F811
    wl = picgen.random_small(70 + ppc, nx=37, nz=11, ppc=ppc, bc_x=ppc % 2, dx=0.5, dz=0.4, dt=0.4,
                             temps=(te, 0.5))
    if keep > 1:
        thin(wl, keep)
    print(f"[gpu-case] grouped ppc={ppc} te={te} keep={keep} tile={tile} ids={ids}", flush=True)
    ctx, orc = setup_both(pic, wl, fields=picgen.random_fields(ppc, wl.grid), tile=tile, track_ids=ids)
    check_moments(ctx, orc)
    ctx.step(2)
    orc.step(2)
    check_fields(ctx, orc)
    check_moments(ctx, orc)
    check_particles(ctx, orc, wl, ids=ids)
    assert ctx.get_info()["overflow_flags"] == 0
    ctx.close()


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,nz,ppc,te", [(39, 1037, 3, 200.0), (16, 1026, 9, 1.0)])
def test_direct_form(pic, nx, nz, ppc, te, bc):  # noqa: F811
    wl = picgen.random_small(90 + ppc, nx=nx, nz=nz, ppc=ppc, bc_x=bc, dx=0.5, dz=0.4, dt=0.4,
                             temps=(te, 0.5))
    print(f"[gpu-case] direct {nx}x{nz} ppc={ppc} te={te} bc={bc}", flush=True)
    ctx, orc = setup_both(pic, wl, fields=picgen.random_fields(3, wl.grid), track_ids=False)
    ctx.step(2)
    orc.step(2)
    check_fields(ctx, orc)
    check_moments(ctx, orc)
    check_particles(ctx, orc, wl, ids=False)
    assert ctx.get_info()["overflow_flags"] == 0
    ctx.close()


@pytest.mark.parametrize("rank", [0, 1, 2])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,nz,ppc,tile", [(37, 29, 5, (0, 0)), (41, 60, 39, (0, 0)),
                                            (41, 60, 40, (0, 0)), (5, 4, 300, (2, 3)),
                                            (341, 6, 6, (64, 2)), (3, 683, 7, (0, 0))])
def test_sort(pic, nx, nz, ppc, tile, bc, rank):  # noqa: F811
    """Cells in two or three scan blocks, the last one ragged; 64 and 16 lanes per cell in the
    ranker, with more slots per cell than it loads ahead."""
    wl = picgen.random_small(120 + ppc, nx=nx, nz=nz, ppc=ppc, bc_x=bc, dx=0.5, dz=0.4, dt=0.4,
                             temps=(200.0, 0.5))
    print(f"[gpu-case] sort {nx}x{nz} ppc={ppc} bc={bc} rank={rank}", flush=True)
    ctx, orc = setup_both(pic, wl, fields=picgen.random_fields(ppc, wl.grid), tile=tile)
    ctx.set_rank_mode(rank)
    ctx.step(3)
    orc.step(3)
    check_moments(ctx, orc)
    check_particles(ctx, orc, wl)
    assert ctx.get_info()["overflow_flags"] == 0
    ctx.close()


@pytest.mark.parametrize("what,mover", [("u", 0), ("h", 0), ("h", 1)])
def test_moments_that_are_not_finite_stay_in_their_cell(pic, what, mover):  # noqa: F811
    """A particle's momentum, or a cell's H, overflows when squared: the four nodes of that cell
    carry it and no others.  (With mover options such a momentum's Lorentz factor is infinite and
    its moments are zero.)"""
    wl = picgen.random_small(131, nx=11, nz=7, ppc=9, bc_x=0, dx=0.5, dz=0.4, dt=0.4)
    sp = wl.species[0]
    n = sp.ux.size // 2
    i, k = int(sp.xi_x[n]), int(sp.xi_z[n])
    e, h = picgen.random_fields(131, wl.grid)
    if what == "u":
        sp.ux[n] = 1e200
    else:
        h[2, k, i] = 1e200
    print(f"[gpu-case] overflowing {what}, mover {mover}", flush=True)
    ctx, _ = setup_both(pic, wl, fields=(e, h))
    if mover:
        ctx.set_mover(mover)
    m = ctx.read_moments()
    bad = ~np.isfinite(m).all(axis=0)
    own = np.zeros_like(bad)
    for dk in (0, 1):
        for di in (0, 1):
            own[(k + dk) % m.shape[1], (i + di) % m.shape[2]] = True
    assert (bad == own).all()
    ctx.close()
