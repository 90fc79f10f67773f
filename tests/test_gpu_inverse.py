"""The dense inverse at the edges of its forms: one workgroup up to 32 and 64 rows,
panels up to 256, 512, 1024, 2048 and 4096 rows, one column at a time above."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    c = mbt.mbt_ctx_create(0)
    yield c
    mbt.mbt_ctx_destroy(c)


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 64, 65, 72, 73, 255, 256, 257, 512, 513, 1024, 1025, 2049])
def test_inverse_at_the_edges_of_its_forms(ctx, n):
    """||X A - 1||_F <= 1e-11 n for a well-conditioned random matrix, a row-permuted
    diagonal (every pivot off the diagonal) at 1e-13 n, there also at
    scales whose squares come near the ends of the range; a zero column is refused."""
    from paper_2608_17844_amd import mbt
    print("n=%d" % n, flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)) + 2 * np.eye(n)
    assert np.linalg.norm(mbt.mbt_dbg_inverse(ctx, A) @ A - np.eye(n)) <= 1e-11 * n
    D = np.zeros((n, n), complex)
    D[np.arange(n), rng.permutation(n)] = (1.0 + rng.random(n)) * 1j
    for scale in (1.0, 1e-150, 1e140):
        X = mbt.mbt_dbg_inverse(ctx, D * scale)
        assert np.linalg.norm((X * scale) @ D - np.eye(n)) <= 1e-13 * n
    A[:, n // 2] = 0.0
    with pytest.raises(mbt.MbtError):
        mbt.mbt_dbg_inverse(ctx, A)
