"""The block products at the widths and block sizes at which their split changes
(row tiles per wave, rounds of column tiles per workgroup, order of a wave's
tiles): every column has the bits that it has in a batch of two."""
import numpy as np
import pytest

from paper_2608_17844_amd import workloads as W

pytestmark = pytest.mark.gpu

WIDTHS = [1, 15, 17, 31, 33, 47, 49, 63, 65, 113, 129, 255, 257, 514, 600, 750, 850, 1023, 1024]


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    h = mbt.mbt_ctx_create(0)
    yield h
    mbt.mbt_ctx_destroy(h)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("M", [1, 7, 9, 15, 17, 31])
def test_columns_keep_their_bits_at_any_width(ctx, M, prec):
    from paper_2608_17844_amd import mbt
    lat, dip = W.Lattice(2, 1, 0.5, 0.5), W.Dipole(0.5, 0.005, M)
    V = W.random_vectors(2 * M, max(WIDTHS), seed=5)
    p = mbt.MBT_FP64 if prec == "f64" else mbt.MBT_FP32
    a = mbt.mbt_array_create_dipole(ctx, dip, lat)
    try:
        for op in (0, 1):
            ref = np.hstack([mbt.mbt_dbg_matvec(ctx, a, 0.93, V[:, j:j + 2], op=op, prec=p)
                             for j in range(0, V.shape[1], 2)])
            for R in WIDTHS:
                y = mbt.mbt_dbg_matvec(ctx, a, 0.93, V[:, :R], op=op, prec=p)
                assert np.array_equal(y, ref[:, :R]), (M, R, op)
        print("M", M, prec, flush=True)
    finally:
        mbt.mbt_array_destroy(a)
