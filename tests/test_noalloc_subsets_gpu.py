"""The no-allocation call of a FP64 context whose k points take different subsets of q (w_kq): a k of fewer but larger pairs
than the one that the work items are chosen for fits the scratch as one item per pair, so it must be served. Against
matrix() (the same plan: the same bits) and the definition.

Tolerance: V sums n_q n_occ products of N_MB terms (v is diagonal here): 4 (n_q n_occ + N_MB) 2^-53 of |A|^H |v| |A|.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_fewer_larger_pairs_fit_the_scratch():
    import paper_1003_0524_amd as lib
    nb, nocc, npw = 128, 3, [640] * 7 + [1739] * 5
    w = np.zeros((2, 12))
    w[0, :7], w[1, 7:] = 1 / 7, 1 / 5
    rng = np.random.default_rng(3)
    diag = [rng.uniform(0.5, 2.0, size=n) for n in npw]
    ex = lib.Exchange([nb, nb], npw, [], nocc, [np.diag(d).astype(complex) for d in diag], [], [], w_kq=w,
                      precision="fp64")
    try:
        for k in range(2):
            qs = [q for q in range(12) if w[k, q]]
            A = [rng.standard_normal((nocc, nb, npw[q])) + 1j * rng.standard_normal((nocc, nb, npw[q])) for q in qs]
            M = torch.from_numpy(np.concatenate([a.ravel() for a in A])).cuda()
            out = torch.empty(nb * nb, dtype=torch.complex128, device="cuda")
            one = ex.matrix_noalloc(k, M, out).cpu().numpy()
            assert np.array_equal(one, ex.matrix(k, M).cpu().numpy())
            ref, scale = np.zeros((nb, nb), complex), np.zeros((nb, nb))
            for a, q in zip(A, qs):
                a = a.transpose(1, 0, 2).reshape(nb, -1)
                d = np.tile(diag[q], nocc) * w[k, q]
                ref -= (a.conj() * d) @ a.T
                scale += (np.abs(a) * d) @ np.abs(a).T
            tol = 4 * (len(qs) * nocc + max(npw)) * 2.0 ** -53 * scale
            assert np.all(np.abs(one - ref) <= tol), np.max(np.abs(one - ref) / tol)
    finally:
        ex.close()
