"""The lattice transforms on every grid shape (each axis 16 to 128 points): the
operator and its adjoint against the dense oracle, on lattices that fill none of
the axes and batches that end inside a group of columns."""
import numpy as np
import pytest

from oracle import mom
from paper_2608_17844_amd import workloads as W

pytestmark = pytest.mark.gpu

SIDES = {8: 7, 16: 11, 32: 21, 64: 37}   # transform length of an axis: elements along it


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    h = mbt.mbt_ctx_create(0)
    yield h
    mbt.mbt_ctx_destroy(h)


@pytest.mark.parametrize("ly", sorted(SIDES))
@pytest.mark.parametrize("lx", sorted(SIDES))
def test_operator_on_grid(ctx, lx, ly):
    from paper_2608_17844_amd import mbt
    lat, dip = W.Lattice(SIDES[lx], SIDES[ly], 0.5, 0.5), W.Dipole(0.5, 0.005, 3)
    print("grid", lx, ly, flush=True)
    a = mbt.mbt_array_create_dipole(ctx, dip, lat)
    try:
        Z = mom.fill_dense(lat, dip, 1.0)
        aZ = np.abs(Z)
        # the rounding bound of the operator test: two transforms and a sum over the bases per value
        c = 16 * (np.log2(4 * lx * ly) + dip.nbases)
        for R in (1, 7):
            x = W.random_vectors(Z.shape[0], R, seed=3)
            for op, ref, mag in ((0, Z @ x, aZ @ np.abs(x)), (1, Z.conj().T @ x, aZ.T @ np.abs(x))):
                for prec, u in ((mbt.MBT_FP64, 2.0 ** -53), (mbt.MBT_FP32, 2.0 ** -24)):
                    y = mbt.mbt_dbg_matvec(ctx, a, 1.0, x, op=op, prec=prec)
                    assert np.all(np.abs(y - ref) <= c * u * mag), (R, op, prec)
    finally:
        mbt.mbt_array_destroy(a)


@pytest.mark.parametrize("nx,ny", [(64, 64), (53, 52), (52, 52), (64, 32), (32, 64)])
def test_operator_by_share_of_the_grid(ctx, nx, ny):
    """The largest grids filled to both sides of the share at which the FP64 inverse
    transform changes the place where its first x-parity waits, and filled whole."""
    from paper_2608_17844_amd import mbt
    lat, dip = W.Lattice(nx, ny, 0.5, 0.5), W.Dipole(0.5, 0.005, 1)
    print("lattice", nx, ny, flush=True)
    a = mbt.mbt_array_create_dipole(ctx, dip, lat)
    try:
        Z = mom.fill_dense(lat, dip, 1.0)
        x = W.random_vectors(Z.shape[0], 3, seed=4)
        c = 16 * (np.log2(4 * 64 * 64) + 1)
        y = mbt.mbt_dbg_matvec(ctx, a, 1.0, x)
        assert np.all(np.abs(y - Z @ x) <= c * 2.0 ** -53 * (np.abs(Z) @ np.abs(x)))
    finally:
        mbt.mbt_array_destroy(a)
