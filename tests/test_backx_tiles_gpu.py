"""The back-transform at the edges of its 16 x 16 tiles and of its quarters of the band index.

Tolerance: an element of Z V Z^H sums n_b^2 complex triple products; |error| <= (8 n_b + 16) 2^-53 |Z| |V| |Z|^H, the
oracle's own rounding included.
"""
import numpy as np
import pytest

from oracle import backx

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 4, 16, 17, 35, 64, 113, 128])
def test_tile_edges(nb):
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(nb)
    ex = lib.Exchange([nb], [7], [], 1, [np.eye(7, dtype=complex)], [], [], precision="fp64")
    try:
        m = rng.standard_normal((nb, 7)) + 1j * rng.standard_normal((nb, 7))
        v = ex.matrix(0, torch.from_numpy(m.ravel()).cuda())
        V = np.asarray(v.cpu().numpy()).reshape(nb, nb)
        for nG in (1, 15, 16, 17, 33, 130):
            Z = rng.standard_normal((nG, nb)) + 1j * rng.standard_normal((nG, nb))
            G = ex.back_transform(0, torch.from_numpy(np.ascontiguousarray(Z.T)).cuda().T).cpu().numpy()
            ref = backx.back_transform(Z, V)
            tol = (8 * nb + 16) * 2.0 ** -53 * np.abs(Z) @ np.abs(V) @ np.abs(Z).T
            assert np.all(np.abs(G - ref) <= tol), (nb, nG)
    finally:
        ex.close()
