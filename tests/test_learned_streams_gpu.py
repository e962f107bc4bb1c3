"""The learned extrapolator's calls in the order of their streams: inputs that queued work is still writing, outputs that
queued work still reads, on the default stream and on another one, and calls of one context on two streams at once.
Against the same calls with a synchronisation between them: the same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NB, NK, NBLK = 24, 6, 8


def _context(n_k):
    import paper_1003_0524_amd as lib
    return lib.Exchange([NB] * n_k, [3], [], 1, [np.eye(3, dtype=complex)], [], [], precision="fp64")


def _hermitian(n_k, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n_k, NB, NB), generator=g, dtype=torch.complex128, device="cuda")
    return [h.contiguous().view(-1) for h in x + x.conj().transpose(1, 2)]


class _Busy:
    """Some tens of milliseconds of work on the current stream."""

    def __init__(self):
        self.a = torch.randn((4096, 4096), dtype=torch.float64, device="cuda")
        self.b = torch.empty_like(self.a)

    def __call__(self):
        for _ in range(20):
            torch.matmul(self.a, self.a, out=self.b)


@pytest.mark.parametrize("own_stream", [False, True])
def test_inputs_still_being_written_and_outputs_still_being_read(own_stream):
    ex, busy = _context(NK), _Busy()
    try:
        ex.nn_init(64, 32, NK * NBLK ** 2, 3)
        V0, V1 = _hermitian(NK, 1), _hermitian(NK, 2)
        P0, P1 = torch.cat(V0), torch.cat(V1)
        Z0 = ex.eigh(V0)[1]
        X0, X1 = torch.randn((4, 64), device="cuda"), torch.randn((4, 64), device="cuda")

        def calls(V, Z, P, X, y, outs, before):
            before()
            w, z = ex.eigh(V)
            before()
            proj = ex.nn_project(V, V0, Z, NBLK, 0.5)
            before()
            x, norm = ex.nn_features(P, P0 * 0.5, 64, 7)
            before()
            pred = ex.nn_predict(X)
            before()
            ex.nn_expand(V, Z, NBLK, y, 0.25, outs)
            return [w, z, proj, x, norm, pred] + outs

        y1 = torch.randn((NK, NBLK * NBLK), device="cuda")
        torch.cuda.synchronize()
        Z1 = ex.eigh(V1)[1]
        torch.cuda.synchronize()
        ref = calls(V1, Z1, P1, X1, y1, [torch.empty_like(v) for v in V0], torch.cuda.synchronize)
        torch.cuda.synchronize()

        # the same inputs written behind queued work, over others
        V, Z, P, X = [v.clone() for v in V0], Z0.clone(), P0.clone(), X0.clone()
        y, outs = torch.zeros_like(y1), [torch.full_like(v, 3.0) for v in V0]
        kept = []

        def late():
            for t, s in [*zip(V, V0), (Z, Z0), (P, P0), (X, X0), (y, 0 * y1)]:
                t.copy_(s)
            busy()
            for t, s in [*zip(V, V1), (Z, Z1), (P, P1), (X, X1), (y, y1)]:
                t.copy_(s)
            kept[:] = [o.clone() for o in outs]                  # reads the outputs before the call may write them

        stream = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            got = calls(V, Z, P, X, y, outs, late)
        torch.cuda.synchronize()
        names = ["w", "Z", "project", "features", "norm", "predict"] + [f"V{k}" for k in range(NK)]
        for name, a, b in zip(names, got, ref):
            assert torch.equal(a, b), name
        assert all(bool((k == 3.0).all()) for k in kept)
    finally:
        ex.close()


def test_default_stream_inputs_of_a_call_on_another_stream():
    """The matrices of a table call come from the default stream's queued work, whatever stream the call is on."""
    ex, busy = _context(NK), _Busy()
    try:
        V0, V1 = _hermitian(NK, 1), _hermitian(NK, 2)
        ref = ex.eigh(V1)
        V = [v.clone() for v in V0]
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        busy()
        for a, b in zip(V, V1):
            a.copy_(b)
        with torch.cuda.stream(s):
            got = ex.eigh(V)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, ref))
    finally:
        ex.close()


def test_two_streams_share_the_tables_in_turn():
    """More matrices than the GPU takes at once: the last ones of a call read the tables while the next call is queued."""
    n_k = 1500
    ex = _context(n_k)
    try:
        sets = [_hermitian(n_k, 10 + i) for i in range(4)]
        ref = [ex.eigh(s) for s in sets]
        torch.cuda.synchronize()
        proj = [ex.nn_project(s, sets[0], r[1], NBLK, 1.0) for s, r in zip(sets, ref)]
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        got, got_p = [], []
        for i, s in enumerate(sets):
            with torch.cuda.stream(streams[i % 2]):
                got.append(ex.eigh(s))
                got_p.append(ex.nn_project(s, sets[0], ref[i][1], NBLK, 1.0))
        torch.cuda.synchronize()
        for i in range(len(sets)):
            assert torch.equal(got[i][0], ref[i][0]) and torch.equal(got[i][1], ref[i][1]), i
            assert torch.equal(got_p[i], proj[i]), i
    finally:
        ex.close()
