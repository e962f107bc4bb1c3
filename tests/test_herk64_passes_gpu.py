"""FP64 Cholesky/HERK kernel where the last n'' pass is short: every instance with several n'' values a pass, numbers of
occupied bands that leave it one or all but one of them, block-sparse rows in the kernel, read from the workspace and
none, every split of the passes and row parts; and systems for which the planner itself picks such a pass. Against the
oracle.

Tolerance: as for the kernel's other tests, 0.25 (n_q n_occ + 2) N_MB 2^-53 of ||A^H v A||.
"""
import os

import numpy as np
import pytest

import synth
from oracle import precision as pr, vx

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

INSTANCES = [(1, 1), (1, 2), (1, 4), (1, 8), (1, 12), (2, 1), (2, 2), (2, 3), (2, 4), (2, 6), (3, 1), (3, 2), (3, 3),
             (3, 4), (4, 1), (4, 2), (5, 1), (8, 1), (9, 1), (13, 1), (16, 1)]
# channel radial counts: chunks of several channels, a channel longer than a chunk (rows through the workspace), none
CHANNELS = {"chunks": [6, 1, 3, 9, 2, 17, 4], "workspace": [19, 3], "none": []}


class _Env:
    def __init__(self, **kw):
        self.kw = kw

    def __enter__(self):
        os.environ.update(self.kw)

    def __exit__(self, *a):
        for k in self.kw:
            os.environ.pop(k, None)


def _system(name, seed, nb, nocc, ch, npw):
    q = np.random.default_rng([seed, 7]).uniform(0.05, 0.95, size=(len(npw), 3))
    return synth.Config(f"passes-{name}", 700 + seed, 0, 9.0 * np.eye(3), q, n_k=len(nb), n_occ=nocc, n_bands=list(nb),
                        ch_nrad=list(ch), n_pw=list(npw))


def _check(cfg, envs, np_dt):
    import paper_1003_0524_amd as lib
    E, D, C = synth.coulomb_blocks(cfg)
    v = [vx.assemble_v(E[q], D, C) for q in range(cfg.n_q)]
    Ms, refs = [], []
    for k in range(cfg.n_k):
        blocks = [synth.m_block(cfg, k, q, np_dt) for q in range(cfg.n_q)]
        refs.append(vx.vx_k([b.astype(np.complex128) for b in blocks], v, cfg.weights_q()))
        Ms.append(torch.from_numpy(np.concatenate([b.ravel() for b in blocks])).cuda())
    tol = 0.25 * (cfg.n_q * cfg.n_occ + 2) * max(cfg.n_mb(q) for q in range(cfg.n_q)) * 2.0 ** -53
    for env, want in envs:
        with _Env(**env):
            ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(),
                              precision="fp64")
        if want:
            assert ex.query(3) == want, (ex.query(3), want)
        V = [x.cpu().numpy() for x in ex.matrix_all(Ms)]
        ex.close()
        for k in range(cfg.n_k):
            err = pr.normwise_error(V[k], refs[k])
            assert err <= tol, (cfg.name, env, k, err, tol)


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("channels", list(CHANNELS))
@pytest.mark.parametrize("nbt,ng", INSTANCES)
def test_short_last_pass(nbt, ng, channels, dt):
    ident = 2000 + 16 * nbt + ng
    for rest in sorted({1, ng - 1} - {0}) if ng > 1 else [2]:
        nocc = 2 * ng + rest if ng > 1 else rest
        cfg = _system(f"{nbt}-{ng}-{channels}-{rest}", nbt * 20 + ng, [8 * nbt - 3], nocc, CHANNELS[channels], [66, 1, 130])
        envs = [({"EXC_HERK64": f"{ident},{p},{g}"}, ident) for p in (0, 1, 2) for g in (1, 2, 0)]
        _check(cfg, envs, np.complex128 if dt == "c128" else np.complex64)


@pytest.mark.parametrize("nb,nocc,n_q,npw", [(13, 7, 64, 13), (24, 5, 64, 13), (8, 11, 64, 20), (31, 13, 8, 303)])
def test_short_last_pass_of_the_planner(nb, nocc, n_q, npw):
    _check(_system(f"planner-{nb}", nb, [nb], nocc, [9, 4, 4, 4, 4, 6, 2], [npw] * n_q), [({}, 0)], np.complex128)
