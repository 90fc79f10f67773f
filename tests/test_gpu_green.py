"""The Green's function of the RWG fill against 80-bit arithmetic: its error is no
larger than that of the plain form (square root, sine and cosine of kR, division),
each operation of which is rounded once, from a hundredth of a radian on."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGES = [0.01, 0.05, 0.2, 0.6, 1.0, 2.0, 6.0, 20.0, 60.0, 200.0]   # of kR


@pytest.fixture(scope="module")
def ctx():
    from paper_2608_17844_amd import mbt
    h = mbt.mbt_ctx_create(0)
    yield h
    mbt.mbt_ctx_destroy(h)


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="needs 80-bit long double")
@pytest.mark.parametrize("i", range(len(EDGES) - 1))
def test_green_error_at_most_the_plain_forms(ctx, i):
    from paper_2608_17844_amd import mbt
    n = 200_000
    rng = np.random.default_rng(i)
    k = 2.0 * np.pi * 0.93
    R2 = (EDGES[i] * (EDGES[i + 1] / EDGES[i]) ** rng.random(n) / k) ** 2
    print("kR from", EDGES[i], "to", EDGES[i + 1], flush=True)
    L = np.longdouble
    four_pi = 16 * np.arctan(L(1))
    R = np.sqrt(L(1) * R2)
    size = 1 / (four_pi * R)
    re, im = np.cos(k * R) * size, -np.sin(k * R) * size
    # the plain form in FP64, sine and cosine rounded from 80 bits
    Rd = np.sqrt(R2)
    x = L(1) * (k * Rd)
    f = (0.25 / np.pi) / Rd
    plain = np.cos(x).astype(np.float64) * f - 1j * (np.sin(x).astype(np.float64) * f)

    def rms(G):
        return float(np.sqrt(np.mean(((G.real - re) ** 2 + (G.imag - im) ** 2) / size ** 2)))

    G = mbt.mbt_dbg_green(ctx, k, R2)
    assert rms(G) <= rms(plain), (rms(G), rms(plain))
