"""Few pairs per k in the fused instances that stream their Gram tiles: every chunk of rows in a slot of its own, added
up in the order of one item per pair: the bits must be those of the no-allocation call, which keeps one item per pair.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (bands per k, n_occ, channel radial counts, plane waves per q)
CASES = {
    "5-tiles": ([37, 13, 25], 5, [3, 2, 9, 1, 4] * 5, [37, 130, 64]),
    "8-tiles": ([64], 3, [5] * 13, [128, 129]),
    "dense only": ([30], 7, [], [191, 64, 1]),
    "10-tiles": ([77], 2, [4] * 7, [100, 65]),
    "16-tiles": ([121], 2, [2] * 40, [60, 200]),
}


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("precision", ["fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("name", list(CASES))
def test_same_bits_as_one_item_per_pair(name, precision, dt):
    import paper_1003_0524_amd as lib
    nb, nocc, ch, npw = CASES[name]
    i = list(CASES).index(name)
    q = np.random.default_rng([9, i]).uniform(0.05, 0.95, size=(len(npw), 3))
    cfg = synth.Config(f"chunks-{i}", 300 + i, 0, 9.0 * np.eye(3), q, n_k=len(nb), n_occ=nocc, n_bands=list(nb),
                       ch_nrad=list(ch), n_pw=list(npw))
    E, D, C = synth.coulomb_blocks(cfg)
    ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(),
                      precision=precision, form="herk", batched=True)
    try:
        np_dt = np.complex128 if dt == "c128" else np.complex64
        for k in range(cfg.n_k):
            m = torch.from_numpy(np.concatenate([synth.m_block(cfg, k, j, np_dt).ravel() for j in range(cfg.n_q)])).cuda()
            one = torch.empty(nb[k] ** 2, dtype=torch.complex128, device="cuda")
            for mask in (False, True):
                if mask:
                    keep = np.ones((nb[k], nb[k]), bool)
                    keep[:8, 8:16] = keep[8:16, :8] = False
                    ex.band_mask(k, keep)
                ref = ex.matrix_noalloc(k, m, one).cpu().numpy()
                got = ex.matrix(k, m).cpu().numpy()
                assert np.array_equal(got, ref), (name, precision, dt, k, mask)
    finally:
        ex.close()
