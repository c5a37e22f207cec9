"""Moments that are not finite stay at the nodes of their particle's cell, in the forms of the
deposit that sum the particles of neighbouring cells together."""
from __future__ import annotations

import numpy as np
import pytest

import picgen
from tests.test_gpu_batch import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


def corner_nodes(m, i, k):
    own = np.zeros(m.shape[1:], dtype=bool)
    for dk in (0, 1):
        for di in (0, 1):
            own[(k + dk) % m.shape[1], (i + di) % m.shape[2]] = True
    return own


def loaded(pic, wl, fields, precision):  # noqa: F811
    ctx = pic.Context(wl.grid, precision=precision)
    ctx.load_fields(*fields)
    for s, sp in enumerate(wl.species):
        ctx.load_particles(s, sp.q, sp.m, sp.w, sp.xi_x, sp.xi_z, sp.ux, sp.uy, sp.uz)
    return ctx


@pytest.mark.parametrize("nx,nz,ppc", [(39, 1037, 3), (16, 1026, 9), (37, 11, 17)])
def test_field_that_overflows_in_32_bits(pic, nx, nz, ppc):  # noqa: F811
    """B = 1e25: B.B is infinite in 32 bits, its reciprocal 0, a0 = 0 is finite and delta-j is
    0 times infinity."""
    wl = picgen.fp32_representable(picgen.random_small(7, nx=nx, nz=nz, ppc=ppc, bc_x=0, dx=0.5, dz=0.4, dt=0.4))
    e, h = picgen.random_fields(7, wl.grid)
    i, k = nx // 2, nz // 2
    h[2, k, i] = 1e25
    print(f"[gpu-case] field overflow, mixed, {nx}x{nz} ppc={ppc}", flush=True)
    ctx = loaded(pic, wl, (e, h), 1)
    m = ctx.read_moments()
    bad = ~np.isfinite(m).all(axis=0)
    assert (bad == corner_nodes(m, i, k)).all()
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("own", [True, False])
def test_current_that_overflows_beside_a_finite_response(pic, precision, own):  # noqa: F811
    """Density times charge overflows, density times charge squared over mass does not (a species'
    constants, made in 64 bits, overflow together); with a density per particle (own) for one
    particle, otherwise for a species of one particle."""
    wl = picgen.random_small(8, nx=13, nz=9, ppc=9, bc_x=0, dx=0.5, dz=0.4, dt=0.4)
    big, q, m = (1e300, 1e9, 1e20) if precision == 0 else (1e30, 1e9, 1e20)
    sp = wl.species[1]
    sp.q, sp.m = q, m
    n = sp.ux.size // 2
    for a in (sp.ux, sp.uy, sp.uz):
        a[:] = 0.5
    i, k = int(sp.xi_x[n]), int(sp.xi_z[n])
    if own:
        sp.w = np.full(sp.ux.size, 1e-30)
        sp.w[n] = big
    else:
        for f in ("xi_x", "xi_z", "ux", "uy", "uz"):
            setattr(sp, f, getattr(sp, f)[n:n + 1].copy())
        sp.w = big
    if precision:
        wl = picgen.fp32_representable(wl)
    print(f"[gpu-case] current overflow, precision {precision}, own densities {own}", flush=True)
    ctx = loaded(pic, wl, picgen.random_fields(8, wl.grid), precision)
    mom = ctx.read_moments()
    bad = ~np.isfinite(mom).all(axis=0)
    assert bad.any() and not (bad & ~corner_nodes(mom, i, k)).any()
    assert np.isfinite(mom[12:]).all() and (np.isfinite(mom[:9]).all() or not (own or precision))
    ctx.close()
