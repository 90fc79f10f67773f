"""Narrow batches: the sweeps over short rows (several vectors per wave, rows
joined in the updates) and the transforms of few columns give each right-hand side
the bits it has in a wide batch, on both sides of every width at which a launch
changes, for 1, 2 and 4 folded rows and row counts that no join divides."""
import numpy as np
import pytest

from paper_2608_17844_amd import workloads as W

pytestmark = pytest.mark.gpu

WIDE = 144


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    h = mbt.mbt_ctx_create(0)
    yield h
    mbt.mbt_ctx_destroy(h)


@pytest.mark.parametrize("prec", ["f64", "mixed"])
@pytest.mark.parametrize("nx,ny,M", [(5, 5, 15), (6, 5, 7), (12, 10, 15), (17, 9, 5)])
def test_narrow_batches_have_the_bits_of_a_wide_one(ctx, nx, ny, M, prec):
    from paper_2608_17844_amd import mbt
    lat, dip = W.Lattice(nx, ny, 0.5, 0.5), W.Dipole(0.5, 0.005, M)
    V = W.random_vectors(nx * ny * M, WIDE, seed=5)
    if prec == "f64":
        opts = mbt.mbt_default_opts(prec=mbt.MBT_FP64, tol=1e-9)
    else:
        opts = mbt.mbt_default_opts(prec=mbt.MBT_FP32, restart=32, inner_tol=1e-3, refine_tol=1e-9, refine_max=8)
    arr = mbt.mbt_array_create_dipole(ctx, dip, lat)
    try:
        ref, iters, _ = mbt.mbt_dbg_solve(ctx, arr, 1.05, opts, V)
        # the sweeps' rows are R, 2R or 4R columns; their launches change at 32 and 64
        for R in (1, 2, 4, 8, 9, 10, 16, 17, 18, 32, 33, 34, 64, 65, 66):
            if prec == "mixed" and R % 2:
                continue   # an odd width keeps the unpacked basis, whose bits differ
            print(nx, ny, M, prec, "R", R, flush=True)
            I, it, _ = mbt.mbt_dbg_solve(ctx, arr, 1.05, opts, V[:, :R])
            assert np.array_equal(I, ref[:, :R]) and np.array_equal(it, iters[:R])
    finally:
        mbt.mbt_array_destroy(arr)
