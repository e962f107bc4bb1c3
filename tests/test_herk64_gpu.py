"""FP64 Cholesky/HERK kernel (herk64.hpp) at the edges of its tiles: every band-tile count, dense
blocks around the 16-k panels and 64-row blocks, n'' counts that leave a last pass short,
block-sparse rows around a panel or none, complex128 and complex64 M; all k in one launch, one
launch per k and one per pair. Against the oracle on the same values.

Tolerance: an element of V is a sum over N = n_q n_occ N_MB products of rows of Y, themselves sums
over at most N_MB products, so the normwise rounding error is at most about (n_q n_occ N_MB + 2 N_MB)
2^-53 ||A^H v A||; the random parts add up like square roots, so a quarter of the bound holds with a
wide margin: 0.25 * (n_q n_occ + 2) N_MB 2^-53.
"""
import numpy as np
import pytest

import synth
from oracle import precision as pr, vx

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (bands per k, n_occ, channel radial counts, plane waves per q)
CASES = {
    "1-band": ([1, 1], 1, [], [1, 15]),
    "1-tile": ([8, 5], 13, [3] * 4, [12, 13]),
    "2-tiles": ([9, 16], 5, [1, 2, 9], [14, 60]),
    "3-tiles": ([24, 17], 3, [4] * 7, [58, 9]),
    "4-tiles": ([25, 32], 3, [17, 2], [62, 63]),
    "5-tiles": ([33], 2, [5] * 13, [3, 52]),
    "6-tiles": ([48, 3], 1, [6] * 3, [125, 126]),
    "7-tiles": ([49], 2, [2] * 16, [48, 49]),
    "8-tiles": ([57, 64], 2, [8] * 9, [120, 55]),
    "9-tiles": ([65], 2, [2], [63, 65]),
    "10-tiles": ([80], 1, [3] * 5, [43, 44]),
    "11-tiles": ([81], 1, [], [64, 128]),
    "12-tiles": ([96, 60], 1, [3] * 16, [1, 17]),
    "13-tiles": ([97, 104], 2, [7] * 11, [53, 70]),
    "14-tiles": ([112], 1, [2, 3], [30, 31]),
    "15-tiles": ([113], 1, [4] * 4, [61, 12]),
    "16-tiles": ([121, 128], 1, [5] * 4, [28, 77]),
}


def _case(name):
    nb, nocc, ch, npw = CASES[name]
    i = list(CASES).index(name)
    q = np.random.default_rng([5, i]).uniform(0.05, 0.95, size=(len(npw), 3))
    return synth.Config(f"herk64-{name}", 200 + i, 0, 9.0 * np.eye(3), q, n_k=len(nb), n_occ=nocc,
                        n_bands=list(nb), ch_nrad=list(ch), n_pw=list(npw))


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("name", list(CASES))
def test_every_route_matches_oracle(name, dt):
    import paper_1003_0524_amd as lib
    cfg = _case(name)
    np_dt = np.complex128 if dt == "c128" else np.complex64
    E, D, C = synth.coulomb_blocks(cfg)
    v = [vx.assemble_v(E[q], D, C) for q in range(cfg.n_q)]
    Ms, refs = [], []
    for k in range(cfg.n_k):
        blocks = [synth.m_block(cfg, k, q, np_dt) for q in range(cfg.n_q)]
        refs.append(vx.vx_k([b.astype(np.complex128) for b in blocks], v, cfg.weights_q()))
        Ms.append(torch.from_numpy(np.concatenate([b.ravel() for b in blocks])).cuda())
    tol = 0.25 * (cfg.n_q * cfg.n_occ + 2) * max(cfg.n_mb(q) for q in range(cfg.n_q)) * 2.0 ** -53
    for route in ("all", "per_k", "per_pair"):
        print(f"[herk64] {name} {dt} {route}", flush=True)
        ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(),
                          precision="fp64", form="herk", batched=route != "per_pair")
        V = ex.matrix_all(Ms) if route != "per_k" else [ex.matrix(k, m) for k, m in enumerate(Ms)]
        V = [x.cpu().numpy() for x in V]
        ex.close()
        for k in range(cfg.n_k):
            err = pr.normwise_error(V[k], refs[k])
            assert err <= tol, (name, dt, route, k, err, tol)
            assert np.array_equal(V[k], V[k].conj().T) and not np.diag(V[k]).imag.any()
