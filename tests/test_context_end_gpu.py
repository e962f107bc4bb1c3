"""After a context's end nothing of it writes into host memory that others have got since; the next contexts, one after
another and in several threads at once, compute what the first did.
"""
import threading
import time

import numpy as np
import pytest

import synth
import test_random_shapes_gpu as shapes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _changed(blocks):
    for b in blocks:
        if b.any():
            return b.nbytes, 4 * int(np.flatnonzero(b)[0])
    return None


def _train(seed):
    import paper_1003_0524_amd as lib
    ex = lib.Exchange([24] * 2, [3], [], 1, [np.eye(3, dtype=complex)], [], [], precision="fp64")
    try:
        rng = np.random.default_rng(seed)
        X, Y = rng.standard_normal((8, 64)).astype(np.float32), rng.standard_normal((8, 128)).astype(np.float32)
        ex.nn_init(64, 32, 128, seed)
        ex.nn_train(X, Y, epochs=20, lr=1e-3)
        return ex.nn_get_params()
    finally:
        ex.close()


def _predict(seed):
    import paper_1003_0524_amd as lib
    ex = lib.Exchange([24] * 2, [3], [], 1, [np.eye(3, dtype=complex)], [], [], precision="fp64")
    try:
        X = np.random.default_rng(seed).standard_normal((8, 64)).astype(np.float32)
        ex.nn_init(64, 32, 128, seed)
        return np.array(ex.nn_predict(X))
    finally:
        ex.close()


def _tuned(cfg):
    import paper_1003_0524_amd as lib
    E, D, C = synth.coulomb_blocks(cfg)
    M = [torch.from_numpy(synth.m_all(cfg, k, np.complex64)).cuda() for k in range(cfg.n_k)]
    ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(), precision="bf16x3",
                      form="herk", batched=True)
    try:
        return [v.cpu().numpy() for v in ex.matrix_all(M)]
    finally:
        ex.close()


@pytest.mark.parametrize("use", ["training", "tuning"])
def test_no_late_writes_after_a_contexts_end(use):
    cfgs = [shapes._cfg(seed) for seed in (3, 4, 4, 4, 5)]
    blocks = []
    for i in range(200):
        if use == "training":
            synth.coulomb_blocks(cfgs[i % 5])        # (a program's own use of the heap between its contexts)
            _train(i)
        else:
            _tuned(cfgs[i % 5])
        time.sleep(0.003)
        # zeroed blocks of the small size classes, taken before the last ones are given back
        blocks = [np.zeros(n // 4, dtype=np.float32) for n in [912] * 24 + list(range(48, 2049, 32)) for _ in range(2)]
        t0 = time.time()
        while time.time() - t0 < 0.006:
            hit = _changed(blocks)
            assert hit is None, f"context {i}: a block of {hit[0]} bytes changed at {hit[1]}"


def test_contexts_after_and_beside_each_other():
    trained = [_train(s) for s in range(4)]
    for s in range(4):
        np.testing.assert_array_equal(_train(s), trained[s])
    want = [_predict(s) for s in range(4)]
    got = [[None] * 6 for _ in want]

    def work(s):
        for i in range(6):
            got[s][i] = _predict(s)

    threads = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s, w in enumerate(want):
        for g in got[s]:
            np.testing.assert_array_equal(g, w)
