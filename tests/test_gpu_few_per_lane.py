"""Mixed runs with few particles per lane, and all mixed members of a batch, add every particle in 64
bits, also on small grids."""
from __future__ import annotations

import numpy as np
import pytest

import picgen
from tests.test_gpu_batch import pic  # noqa: F401  -- fixture

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("labels", [True, False])
@pytest.mark.parametrize("nx,nz,slab,ppc,tile,batch", [
    (64, 64, 64, 4, (0, 0), False), (32, 9, 1, 60, (0, 0), False), (33, 8, 2, 33, (0, 0), False),
    (20, 17, 20, 7, (4, 4), False), (40, 8, 40, 20, (0, 0), False), (64, 64, 64, 4, (0, 0), True),
    (33, 8, 2, 33, (0, 0), True), (40, 8, 40, 65, (0, 0), True), (20, 17, 5, 128, (4, 4), True),
    (130, 9, 130, 5, (0, 0), True), (70, 9, 70, 17, (0, 0), True)])
def test_densities_are_sums_in_64_bits(pic, nx, nz, slab, ppc, tile, batch, labels):  # noqa: F811
    """Offsets in sixteenths and a density of 16 bits: every particle's share of a node is exact in
    32 bits, sums of a few are not.  At rest without fields nothing moves, so the density planes
    after the load (if it takes that form) and after a cycle are the exact sums."""
    print(f"[gpu-case] few per lane {nx}x{nz} slab {slab} ppc={ppc} tile={tile} labels {labels} batch {batch}", flush=True)
    w = 1.0 + 2.0 ** -15
    rng = np.random.default_rng(nx + ppc)
    ci = np.tile(np.repeat(np.arange(nx // 2 - slab // 2, nx // 2 - slab // 2 + slab), ppc), nz)
    ck = np.repeat(np.arange(nz), slab * ppc)
    n = ci.size
    x, z = ci + rng.integers(0, 16, n) / 16.0, ck + rng.integers(0, 16, n) / 16.0
    g = picgen.Grid(nx=nx, nz=nz, dx=0.5, dz=0.5, dt=0.25, bc_x=picgen.BC_PERIODIC, n_species=1,
                    precision=picgen.PREC_MIXED)
    zero = np.zeros(n)
    ctx = pic.Context(g, precision=1, tile=tile, track_ids=labels)
    ctx.load_fields(np.zeros(3 * nx * nz), np.zeros(3 * nx * nz))
    ctx.load_particles(0, -1.0, 1.0, w, x, z, zero, zero, zero)
    want = np.zeros((nz, nx))
    fx, fz = x - ci, z - ck
    for dx, dz, wt in ((0, 0, (1 - fx) * (1 - fz)), (1, 0, fx * (1 - fz)), (0, 1, (1 - fx) * fz), (1, 1, fx * fz)):
        np.add.at(want, ((ck + dz) % nz, (ci + dx) % nx), wt * w)
    b = None
    if batch:
        b = pic.Batch(0, 1)
        b.add(ctx)
    for cycles in ((1, 2) if batch else (0, 1)):
        (b or ctx).step(cycles)
        got = ctx.read_moments()[12]
        assert np.array_equal(got, want), f"after {cycles} cycles off by {np.abs(got - want).max():.2e}"
    if b:
        b.close()
    ctx.close()
