"""Calls of different k of one context on several streams where they share buffers: the block-sparse workspace (FP64 with a
channel longer than the kernel's chunks, the GEMM form, the unfused reduced-precision path) and the buffers of the unbatched
GEMM form; and back-transforms, which share T = Z V. Against the same calls with a synchronisation after each: the same bits.
"""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N_K, NB, NPW, CH, NOCC = 4, [30, 17, 24, 9], [90, 61, 120], [19, 3, 8, 1, 5] * 3, 5


@pytest.mark.parametrize("name,precision,form,batched", [
    ("workspace fp64", "fp64", "herk", True), ("per pair fp64", "fp64", "herk", False),
    ("gemm", "fp64", "gemm", True), ("plain gemm", "fp64", "gemm", False),
    ("tile fp32", "fp32", "herk", True), ("tile bf16x3", "bf16x3", "herk", True)])
def test_streams_in_turn(name, precision, form, batched):
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(4)
    E = []
    for n in NPW:
        m = n + len(CH)
        x = (rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))) / np.sqrt(8 * m)
        E.append(x @ x.conj().T + np.eye(m))
    D = [1.5 * np.eye(b - 1, dtype=complex) for b in CH]
    C = [0.1 * rng.standard_normal(b - 1) + 0.05j for b in CH]
    if precision != "fp64":
        os.environ["EXC_FUSED"] = "0"
    try:
        ex = lib.Exchange(NB, NPW, CH, NOCC, E, D, C, precision=precision, form=form, batched=batched)
    finally:
        os.environ.pop("EXC_FUSED", None)
    try:
        nmb = sum(n + sum(CH) for n in NPW)
        g = torch.Generator(device="cuda").manual_seed(1)
        Ms = [torch.randn(NOCC * nb * nmb, generator=g, dtype=torch.complex128, device="cuda") for nb in NB]
        ref = []
        for k in range(N_K):
            ref.append(ex.matrix(k, Ms[k]).clone())
            torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(N_K)]
        got = []
        for i in range(8):
            for k in range(N_K):
                with torch.cuda.stream(streams[(k + i) % N_K]):
                    got.append((k, ex.matrix(k, Ms[k])))
        torch.cuda.synchronize()
        for k, v in got:
            assert torch.equal(v, ref[k]), (name, k)
    finally:
        ex.close()


def test_back_transforms_in_turn():
    import paper_1003_0524_amd as lib
    rng = np.random.default_rng(8)
    nb, n_G = [100, 60, 100], 1500
    x = rng.standard_normal((40, 40)) + 1j * rng.standard_normal((40, 40))
    ex = lib.Exchange(nb, [40], [], 2, [x @ x.conj().T + np.eye(40)], [], [], precision="fp64")
    try:
        g = torch.Generator(device="cuda").manual_seed(5)
        Zs = []
        for k, b in enumerate(nb):
            ex.matrix(k, torch.randn(2 * b * 40, generator=g, dtype=torch.complex128, device="cuda"))
            Zs.append(torch.randn((b, n_G), generator=g, dtype=torch.complex128, device="cuda").T)
        torch.cuda.synchronize()
        ref = []
        for k in range(3):
            ref.append(ex.back_transform(k, Zs[k]).clone())
            torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(3)]
        got = []
        for i in range(6):
            for k in range(3):
                with torch.cuda.stream(streams[(k + i) % 3]):
                    got.append((k, ex.back_transform(k, Zs[k])))
        torch.cuda.synchronize()
        for k, v in got:
            assert torch.equal(v, ref[k]), k
    finally:
        ex.close()
