"""When a call of few pairs goes through their row chunks: never where that splits nothing, otherwise in the instances that
stream their Gram tiles; in one batch of pairs or several; with the bits of one item per pair.
"""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _context(nb, npw, ch, nocc, precision):
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(7)
    E = []
    for n in npw:
        x = (rng.standard_normal((len(ch) + n,) * 2) + 1j * rng.standard_normal((len(ch) + n,) * 2)) / np.sqrt(8 * (len(ch) + n))
        E.append(x @ x.conj().T + np.eye(len(ch) + n))
    D = [1.5 * np.eye(b - 1, dtype=complex) for b in ch]
    C = [0.1 * rng.standard_normal(b - 1) + 0.05j for b in ch]
    return lib.Exchange([nb], npw, list(ch), nocc, E, D, C, precision=precision)


def _both(ex, nb, npw, ch, nocc, dt=torch.complex128):
    g = torch.Generator(device="cuda").manual_seed(2)
    M = torch.randn(nocc * nb * sum(n + sum(ch) for n in npw), generator=g, dtype=dt, device="cuda")
    V = ex.matrix(0, M).clone()
    batches = int(ex.query(20))
    one = ex.matrix_noalloc(0, M, torch.empty(nb * nb, dtype=torch.complex128, device="cuda"))
    assert torch.equal(V, one)
    return batches


@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6", "fp32"])
@pytest.mark.parametrize("npw,nocc", [([20], 1), ([64, 63, 1], 1), ([40] * 5, 1)])
def test_nothing_to_split(npw, nocc, precision):
    for nb in (64, 80, 128):
        ex = _context(nb, npw, (), nocc, precision)
        try:
            assert _both(ex, nb, npw, (), nocc) == 0
        finally:
            ex.close()


def test_no_room_is_remembered():
    """230 pairs of 10 300 passes, a slot each: 350 GB, more than the card has. The call falls back to one item per pair,
    and the next one does not ask again."""
    nb, nocc, npw = 128, 10300, [1] * 230
    os.environ["EXC_CHUNK_BYTES"] = str(1 << 50)
    try:
        ex = _context(nb, npw, (), nocc, "bf16x3")
    finally:
        del os.environ["EXC_CHUNK_BYTES"]
    try:
        slot = 136 * 256 * 4 + 64 * 16 * 8
        assert len(npw) * nocc * slot > torch.cuda.mem_get_info()[1]
        assert _both(ex, nb, npw, (), nocc, torch.complex64) == 0
        assert ex.query(21) == 1
        assert _both(ex, nb, npw, (), nocc, torch.complex64) == 0
        assert ex.query(21) == 1
    finally:
        ex.close()


# (bands, plane waves, channels, n_occ, bytes that hold the largest pair's slots but not all pairs'): instances of 13 and
# 16 band tiles
CASES = {"80 bands": (80, [130, 64, 191, 40], [4] * 12, 4, 2 << 20), "100 bands": (100, [200] * 6, [3] * 9, 3, 4 << 20),
         "128 bands": (128, [60, 129], [2] * 40, 5, 5 << 20)}


@pytest.mark.parametrize("dt", ["c128", "c64"])
@pytest.mark.parametrize("precision", ["bf16x3", "bf16x6", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_one_batch_and_several(name, precision, dt):
    nb, npw, ch, nocc, few = CASES[name]
    tdt = torch.complex128 if dt == "c128" else torch.complex64
    seen = {}
    for limit in (None, few):
        if limit:
            os.environ["EXC_CHUNK_BYTES"] = str(limit)
        try:
            ex = _context(nb, npw, ch, nocc, precision)
        finally:
            os.environ.pop("EXC_CHUNK_BYTES", None)
        try:
            assert ex.query(16) == 1                     # an instance that streams its Gram tiles
            seen[limit] = _both(ex, nb, npw, ch, nocc, tdt)
        finally:
            ex.close()
    assert seen[None] == 1 and seen[few] >= 2, seen
