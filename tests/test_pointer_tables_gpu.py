"""Calls that change their buffers from one to the next: the device tables of pointers are written in stream order, so
each call must see its own buffers, on one stream and on several, and a captured call the ones that it was captured
with. Against the same calls with a synchronisation after each: the same bits.
"""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _setup(precision):
    import paper_1003_0524_amd as lib
    cfg = synth.make_config("ragged")
    E, D, C = synth.coulomb_blocks(cfg)
    ex = lib.Exchange(cfg.n_bands, cfg.n_pw, cfg.ch_nrad, cfg.n_occ, E, D, C, w_q=cfg.weights_q(), precision=precision)
    base = [torch.from_numpy(synth.m_all(cfg, k)).cuda() for k in range(cfg.n_k)]
    sets = [[m * (1.0 + 0.25 * i) for m in base] for i in range(6)]
    torch.cuda.synchronize()
    return cfg, ex, sets


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_new_buffers_every_call(precision):
    cfg, ex, sets = _setup(precision)
    try:
        ref = []
        for Ms in sets:
            ref.append([ex.matrix(k, m).clone() for k, m in enumerate(Ms)])
            torch.cuda.synchronize()
        outs = [[ex.matrix(k, m) for k, m in enumerate(Ms)] for Ms in sets]          # no wait between them
        torch.cuda.synchronize()
        for o, r in zip(outs, ref):
            assert all(torch.equal(a, b) for a, b in zip(o, r))
        # one k per stream, in turn
        streams = [torch.cuda.Stream() for _ in range(cfg.n_k)]
        outs = []
        for Ms in sets:
            row = []
            for k, m in enumerate(Ms):
                with torch.cuda.stream(streams[k]):
                    row.append(ex.matrix(k, m))
            outs.append(row)
        torch.cuda.synchronize()
        for o, r in zip(outs, ref):
            assert all(torch.equal(a, b) for a, b in zip(o, r))
    finally:
        ex.close()


def test_captured_call_keeps_its_buffers():
    cfg, ex, sets = _setup("fp64")
    try:
        m, nb = sets[0][1], cfg.n_bands[1]
        out = torch.empty(nb * nb, dtype=torch.complex128, device="cuda")
        ref = ex.matrix(1, m, out=out).clone()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ex.matrix(1, m, out=out)
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(nb, nb).T, ref)
    finally:
        ex.close()
