"""The RWG fill where its split of the work changes: meshes of 2 to 128 triangles
(one chunk of test triangles to many, ragged last ones) on lattices with no far
offset, far offsets along one axis, and both, against the oracle's blocks."""
import numpy as np
import pytest

from oracle import rwg
from paper_2608_17844_amd import workloads as W

pytestmark = pytest.mark.gpu

# Rounding relative to the block's largest entry, triangles of size h >= 1/128 wavelength: the charge terms of
# a basis pair cancel to (k h)^2 ~ 1/400 of their size, so far blocks (both sides the same sums of ~50 terms)
# agree to 400 * 50 * 2^-53 ~ 2e-12; the closed form at points a wavelength away cancels by another
# 2 / h^2 ~ 3e4 between its edge terms.
FAR_TOL, NEAR_TOL = 1e-10, 1e-6


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    h = mbt.mbt_ctx_create(0)
    yield h
    mbt.mbt_ctx_destroy(h)


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 4), (5, 1), (3, 3)])
@pytest.mark.parametrize("nseg,nacross", [(2, 1), (2, 3), (18, 1), (64, 1)])
def test_blocks_of_strips(ctx, nseg, nacross, nx, ny):
    from paper_2608_17844_amd import mbt
    mesh = W.strip_mesh(nseg=nseg, nacross=nacross)
    el = rwg.rwg_element(mesh)
    lat = W.Lattice(nx, ny, 0.6, 0.3)
    print("triangles", len(mesh.triangles), "lattice", nx, ny, flush=True)
    a = mbt.mbt_array_create_rwg(ctx, mesh, lat)
    try:
        T = mbt.mbt_dbg_fill_blocks(ctx, a, 1.0, lat, el.M)
        again = mbt.mbt_dbg_fill_blocks(ctx, a, 1.0, lat, el.M)
        assert T.tobytes() == again.tobytes()
        for oy in sorted({-(ny - 1), -1, 0, 1, ny - 1} & set(range(1 - ny, ny))):
            for ox in sorted({-(nx - 1), -1, 0, 2, nx - 1} & set(range(1 - nx, nx))):
                ref = rwg.offset_block(el, lat, 1.0, ox, oy)
                near = abs(ox) <= 1 and abs(oy) <= 1
                err = np.abs(T[oy + ny - 1, ox + nx - 1] - ref).max() / np.abs(ref).max()
                assert err <= (NEAR_TOL if near else FAR_TOL), (ox, oy, err)
    finally:
        mbt.mbt_array_destroy(a)
