"""Block-sparse rows formed on the FP64 matrix cores (the larger FP32 instances of the fused kernel, the wide kernel
above 8 band tiles) at the edges of their units: channels of one function to a whole chunk, groups of 16 rows that end
inside a channel, more than eight multipole rows in a group, chunks of a few rows, complex128 and complex64 M. Against
the oracle.

Tolerance: the FP64 kernel's bound (an element of V sums N = n_q n_occ N_MB products of rows, each a sum over at most
N_MB products; a quarter of the bound for random parts) with the unit roundoff of FP32, 2^-24, and another 2 N_MB for
the inputs rounded to FP32 before their products: 0.25 (n_q n_occ + 4) N_MB 2^-24.
"""
import numpy as np
import pytest

import synth
from oracle import precision as pr, vx

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CHANNELS = {
    "one row": [1],
    "ones": [1] * 40,
    "long": [64, 17, 16, 33],
    "mixed": [16, 17] + [1] * 12 + [30, 5, 4, 4, 8, 9],
    "fives": [5] * 13,
}


@pytest.mark.parametrize("nb,cfg_id,dt", [(40, 121, "c128"), (40, 121, "c64"), (77, 123, "c128"), (100, 180, "c64")])
@pytest.mark.parametrize("name", list(CHANNELS))
def test_rows_match_oracle(name, nb, cfg_id, dt, monkeypatch):
    import paper_1003_0524_amd as lib
    monkeypatch.delenv("EXC_FUSED", raising=False)
    monkeypatch.delenv("EXC_TUNE_CACHE", raising=False)
    monkeypatch.setenv("EXC_FUSED_CFG", str(cfg_id))
    i = list(CHANNELS).index(name)
    q = np.random.default_rng([17, i]).uniform(0.05, 0.95, size=(2, 3))
    cfg = synth.Config(f"rows-{i}-{nb}", 400 + i, 0, 9.0 * np.eye(3), q, n_k=1, n_occ=2, n_bands=[nb],
                       ch_nrad=list(CHANNELS[name]), n_pw=[30, 41])
    np_dt = np.complex128 if dt == "c128" else np.complex64
    E, D, C = synth.coulomb_blocks(cfg)
    blocks = [synth.m_block(cfg, 0, j, np_dt) for j in range(cfg.n_q)]
    ref = vx.vx_k([b.astype(np.complex128) for b in blocks], [vx.assemble_v(E[j], D, C) for j in range(cfg.n_q)],
                  cfg.weights_q())
    ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(), precision="fp32",
                      form="herk", batched=True)
    try:
        V = ex.matrix_all([torch.from_numpy(np.concatenate([b.ravel() for b in blocks])).cuda()])[0].cpu().numpy()
        assert int(ex.query(3)) == cfg_id
        tol = 0.25 * (cfg.n_q * cfg.n_occ + 4) * max(cfg.n_mb(j) for j in range(cfg.n_q)) * 2.0 ** -24
        err = pr.normwise_error(V, ref)
        assert err <= tol, (name, nb, cfg_id, dt, err, tol)
    finally:
        ex.close()
