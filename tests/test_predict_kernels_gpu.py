"""Kernels of a prediction at their edges, against the float64 references: the forward pass around the layer
kernel for few samples (at most 16, layers of a multiple of 256 inputs), the sketch at row counts that do not divide
a workgroup, the expansion at block sizes from one band to all.

Tolerances: the forward pass may be off by the rounding of sums of K FP32 products, (K + 3) 2^-24 times the sum of
the products' magnitudes, and of tanhf (four units), carried through the layers by the magnitudes of their weights;
the sketch by the FP64 rounding of a sum of D terms and that of its FP32 result; the expansion by the FP64 rounding
of two sums over n_blk complex products, (8 n_blk + 8) 2^-53 times the magnitudes summed.
"""
import numpy as np
import pytest

import synth
from oracle import learned as ol
from oracle import mlp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1003_0524_amd as lib
    cfg = synth.make_config("ragged")
    E, D, C = synth.coulomb_blocks(cfg)
    ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(),
                      precision="fp64", form="herk", batched=True)
    yield cfg, ex
    ex.close()


@pytest.mark.parametrize("n", [1, 2, 16, 17])
@pytest.mark.parametrize("I,H,O", [(64, 256, 1), (256, 256, 79), (512, 512, 64), (256, 100, 17), (7, 256, 129)])
def test_forward(ctx, I, H, O, n):
    _, ex = ctx
    ex.nn_init(I, H, O, seed=I + H + O)
    rng = np.random.default_rng([I, H, O, n])
    theta = ex.nn_get_params()
    theta += 0.1 * rng.standard_normal(theta.size).astype(np.float32)          # (biases too)
    ex.nn_set_params(theta)
    th = theta.astype(np.float64)
    X = rng.standard_normal((n, I)).astype(np.float32)
    yr, _ = mlp.forward(th, X.astype(np.float64), I, H, O)
    u = 2.0 ** -24
    x, e, o = np.abs(X.astype(np.float64)), np.zeros((n, I)), 0
    full = X.astype(np.float64)
    for li, (a, b) in enumerate(((I, H), (H, H), (H, O))):
        W, bias = th[o:o + a * b].reshape(b, a), th[o + a * b:o + a * b + b]
        o += a * b + b
        e = e @ np.abs(W).T + (a + 3) * u * (x @ np.abs(W).T + np.abs(bias)) + (4 * u if li < 2 else 0.0)
        full = full @ W.T + bias
        if li < 2:
            full = np.tanh(full)
        x = np.abs(full) + e
    assert np.allclose(full, yr, rtol=1e-12, atol=1e-12)                       # (the layout assumed above)
    yd = ex.nn_predict(torch.from_numpy(X).cuda()).cpu().numpy()
    assert np.all(np.abs(yd - yr) <= e)
    assert np.array_equal(ex.nn_predict(X), yd)


@pytest.mark.parametrize("m", [1, 3, 100, 128])
@pytest.mark.parametrize("D", [1, 2048, 2049, 9001])
def test_sketch(ctx, m, D):
    _, ex = ctx
    rng = np.random.default_rng([m, D])
    a, b = rng.standard_normal(D), rng.standard_normal(D)
    x, nrm = ex.nn_features(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), m, 99)
    s_ref, n_ref = ol.sketch(a - b, m, 99, synth.splitmix64_stream)
    assert abs(nrm.item() - n_ref) <= D * 2.0 ** -53 * n_ref + 2.0 ** -52 * n_ref
    assert np.all(np.abs(x.cpu().numpy() - s_ref) <= 2.0 ** -23 * np.abs(s_ref) + 4 * D ** 1.5 * 2.0 ** -53)


@pytest.mark.parametrize("n_blk", [1, 3, "all"])
def test_expand(ctx, n_blk):
    cfg, ex = ctx
    nbk = min(cfg.n_bands) if n_blk == "all" else n_blk
    rng = np.random.default_rng(nbk)
    V0, Bs = [], []
    for nb in cfg.n_bands:
        A = rng.standard_normal((nb, nb)) + 1j * rng.standard_normal((nb, nb))
        V0.append(A + A.conj().T)
        Bs.append(np.linalg.qr(A)[0])
    y = rng.standard_normal((cfg.n_k, nbk * nbk)).astype(np.float32)
    Z = torch.from_numpy(np.concatenate([b.T.ravel() for b in Bs])).cuda()     # column-major, k by k
    anc = [torch.from_numpy(np.ascontiguousarray(v.T).ravel()).cuda() for v in V0]
    outs = [torch.empty_like(v) for v in anc]
    ex.nn_expand(anc, Z, nbk, torch.from_numpy(y).cuda(), 0.25, outs)
    for k, nb in enumerate(cfg.n_bands):
        B = Bs[k][:, :nbk]
        got = outs[k].cpu().numpy().reshape(nb, nb).T
        ref = ol.expand(V0[k], B, y[k].astype(np.float64), 0.25)
        yk = np.abs(y[k].astype(np.float64).reshape(nbk, nbk))
        mag = np.abs(V0[k]) + 0.25 * 2.0 * np.abs(B) @ (yk + yk.T) @ np.abs(B).T
        assert np.all(np.abs(got - ref) <= (8 * nbk + 8) * 2.0 ** -53 * mag)
