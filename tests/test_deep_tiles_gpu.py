"""The deep variants of the 128x64 / 64x128, 128x128 and 256x128 / 128x256
tiles against the oracle, through the library's own choice: reductions of
fewer steps than stages up to several rounds of them, partial last steps,
shifted edge tiles, both products and the prologue."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_12645_amd import datagen as D
from paper_2006_12645_amd import gba

import gpu_util as U

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(monkeypatch, M, N, K, layout, K2, prologue, tile):
    print("CASE", M, N, K, layout, K2, prologue, flush=True)
    la, lb = D.LAYOUT_NAMES[layout]
    assert gba.select_tile(M, N, K + K2, la, lb) in tile, "not the tile this case is about"
    A, B, bias = D.random_problem(71000 + M + K, M, N, K)
    kw, okw = {}, {}
    if K2:
        P, Q, _ = D.random_problem(72000 + M + K, M, N, K2)
        kw.update(P=U.device_operand(P, la, 8), Q=U.device_operand(Q, lb, 8), second="sub")
        okw.update(second=-1, p_store=D.store(P, D.ROW), q_store=D.store(Q, D.COL), K2=K2)
    with U.recorded_plans(monkeypatch) as plans:
        out = gba.fused_gemm(U.device_operand(A, la, 8), U.device_operand(B, lb, 8), bias=torch.from_numpy(bias).cuda(),
                             act="relu", prologue="relu" if prologue else None, **kw)
    torch.cuda.synchronize()
    assert plans[0]["path"] == "deep", plans
    rows = np.unique(np.concatenate([np.arange(40), np.arange(M - 300, M)]))
    ref = O.fused(D.store(A, D.ROW), D.ROW, D.store(B, D.COL), D.COL, M, N, K, bias=bias, act=O.ACT_RELU,
                  prologue_relu=prologue, rows=rows, **okw)
    U.assert_close(out.cpu().numpy()[rows], ref, what=f"{M}x{N}x{K}+{K2} {layout}")


PRODUCTS = [(False, False), (True, False), (False, True), (True, True)]  # prologue, second product


@pytest.mark.parametrize("prologue,second", PRODUCTS)
@pytest.mark.parametrize("layout", ["RR", "RC", "CC"])
@pytest.mark.parametrize("M,N,K", [(1000, 1400, 392), (2000, 960, 712)])
def test_half(monkeypatch, M, N, K, layout, prologue, second):
    check(monkeypatch, M, N, K - 72 if second else K, layout, 72 if second else 0, prologue, (5, 7))


@pytest.mark.parametrize("prologue,second", PRODUCTS)
@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K", [(1992, 1800, 400), (2048, 2040, 968)])
def test_square(monkeypatch, M, N, K, layout, prologue, second):
    check(monkeypatch, M, N, K - 136 if second else K, layout, 136 if second else 0, prologue, (4,))


@pytest.mark.parametrize("prologue,second", PRODUCTS)
@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K", [(4000, 1920, 2056)])
def test_wide(monkeypatch, M, N, K, layout, prologue, second):
    check(monkeypatch, M, N, K - 520 if second else K, layout, 520 if second else 0, prologue, (2, 3))
