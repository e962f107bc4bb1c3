"""The dense Cholesky of the Coulomb blocks at the edges of its 64-column blocks and 16-column sub-blocks: several q
of different order in one context, the factor seen through V = -sum_q w_q A^H (L L^H) A, and the pivot that a matrix
that is not positive definite is refused at.

Tolerance: the computed factor of an n x n block satisfies |E - L L^H| <= c (n + 1) 2^-53 |L| |L|^H with c = 8 for
complex products; a sub-block's inverse instead of substitution brings in that block's condition, below 4 for these
matrices (unit diagonal weight against small off-diagonal parts): c = 32; the products of V add 4 (n + 2) more.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _pd(n, rng):
    x = (rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))) / np.sqrt(8.0 * max(1, n))
    return x @ x.conj().T + np.eye(n)


@pytest.mark.parametrize("orders", [[1, 2, 15, 16, 17], [63, 64, 65, 1], [127, 128, 129, 48], [321, 200, 3, 256, 79]])
def test_factor_of_several_q(orders):
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(orders)
    E = [_pd(n, rng) for n in orders]
    nb = 5
    ex = lib.Exchange([nb], orders, [], 1, E, [], [], precision="fp64")
    try:
        A = [rng.standard_normal((nb, n)) + 1j * rng.standard_normal((nb, n)) for n in orders]
        V = ex.matrix(0, torch.from_numpy(np.concatenate([a.ravel() for a in A])).cuda())
        V = np.asarray(V.cpu().numpy() if hasattr(V, "cpu") else V).reshape(nb, nb)
        ref, tol = np.zeros((nb, nb), complex), 0.0
        for e, a, n in zip(E, A, orders):
            L = np.abs(np.linalg.cholesky(e))
            ref -= a.conj() @ e @ a.T / len(orders)
            tol = tol + (36 * n + 72) * 2.0 ** -53 * np.abs(a) @ (L @ L.T) @ np.abs(a).T / len(orders)
        err = min(np.max(np.abs(V - ref) / tol), np.max(np.abs(V - ref.T) / tol))
        assert err <= 1.0, err
    finally:
        ex.close()


@pytest.mark.parametrize("at", [0, 15, 16, 47, 63, 64, 100, 128, 149])
def test_refused_at_the_first_bad_pivot(at):
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(at)
    E = [_pd(150, rng), _pd(150, rng)]
    L = np.linalg.cholesky(E[1])
    E[1][at, at] -= np.abs(L[at, at]) ** 2 + 0.5                 # the Schur complement at this pivot: -0.5
    E[1][149, 149] -= 10.0 if at < 149 else 0.0                  # (a later one does not count)
    with pytest.raises(lib.ExchangeError) as e:
        lib.Exchange([4], [150, 150], [], 1, E, [], [], precision="fp64")
    assert e.value.status == -4 or "positive definite" in str(e.value)
    assert f"at q = 1 (pivot {at + 1})" in str(e.value)
