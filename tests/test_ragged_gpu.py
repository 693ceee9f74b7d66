"""Large requests outside the aligned fast path (odd sizes, odd leading
dimensions) against the oracle, on each block tile of the kernel that takes
them: whole and partial last steps of both products, edge tiles shifted by
odd amounts, every layout, both accumulations, a bias at an odd address.  Each
case asserts the tile it is about.  The output is a window of a larger buffer
whose surroundings must stay untouched."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_12645_amd import datagen as D
from paper_2006_12645_amd import gba

import gpu_util as U

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(monkeypatch, want, M, N, K, layout, K2=0, second="sub", prologue=None, bias="row", act="none", accum="f32",
          pad=1, seed=0, rows=None):
    print("CASE", M, N, K, layout, K2, second, prologue, bias, act, accum, pad, flush=True)
    A, B, row = D.random_problem(66000 + seed, M, N, K)
    b = row if bias == "row" else D.uniform_f16(67000 + seed, (M, N))
    la, lb = D.LAYOUT_NAMES[layout]
    kw, okw = {}, {}
    if K2:
        P, Q, _ = D.random_problem(68000 + seed, M, N, K2)
        kw.update(P=U.device_operand(P, la, pad), Q=U.device_operand(Q, lb, pad), second=second)
        okw.update(second=1 if second == "add" else -1, p_store=D.store(P, D.ROW), q_store=D.store(Q, D.COL), K2=K2)
    around = torch.full((M + 2, N + 3), 7.0, dtype=torch.float16, device="cuda")
    out = around[1:M + 1, 1:N + 1]
    with U.recorded_plans(monkeypatch) as plans:
        gba.fused_gemm(U.device_operand(A, la, pad), U.device_operand(B, lb, pad), prologue=prologue, act=act,
                       accum=accum, bias=U.misaligned(b), bias_op="sub", out=out, **kw)
    torch.cuda.synchronize()
    got_plan = plans[0]["path"] if plans[0]["path"] != "unaligned" else plans[0]["bm"]
    assert got_plan == want, plans
    if rows is None:
        rows = np.concatenate([np.arange(min(M, 70)), np.arange(max(0, M - 270), M), [M // 2]])
    rows = np.unique(rows)
    ref = O.fused(D.store(A, D.ROW), D.ROW, D.store(B, D.COL), D.COL, M, N, K, prologue_relu=prologue == "relu",
                  act={"none": O.ACT_NONE, "relu": O.ACT_RELU}[act], bias=b, bias_sign=-1, rows=rows,
                  acc16=accum == "f16", **okw)
    U.assert_close(out.cpu().numpy()[rows], ref, accum=accum, what=f"{M}x{N}x{K} {layout}")
    out.fill_(7.0)
    assert bool((around == 7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [(64, 64, 64, 0), (65, 127, 65, 0), (67, 129, 127, 64), (190, 71, 191, 129),
                                      (513, 66, 321, 0)])
def test_64x64_tile(monkeypatch, M, N, K, K2, layout):
    check(monkeypatch, 64, M, N, K, layout, K2, prologue="relu" if K2 else None, bias="full" if K2 else "row", seed=M)


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2,pad", [(1793, 1665, 65, 0, 1), (1665, 1857, 128, 70, 2), (1536, 1536, 200, 0, 4)])
def test_128x128_tile(monkeypatch, M, N, K, K2, pad, layout):
    check(monkeypatch, 128, M, N, K, layout, K2, second="add", prologue="relu" if K2 else None, act="relu", pad=pad,
          seed=M)


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [(4001, 4095, 641, 0), (4095, 4087, 449, 258)])
def test_256x256_tile(monkeypatch, M, N, K, K2, layout):
    """(Sampled rows: of the first tiles, of both sides of the last tile row's
    edge, whose outputs two workgroups compute, and the last.)"""
    rows = np.r_[:5, 126:130, 254:259, M // 2, M - 258:M - 254, M // 256 * 256 - 2:M // 256 * 256 + 2, M - 5:M]
    check(monkeypatch, 256, M, N, K, layout, K2, prologue="relu" if K2 else None, bias="full" if K2 else "row", seed=M,
          rows=rows)


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2,want", [
    (75, 133, 288, 0, 64), (131, 66, 160, 64, 64), (1793, 1665, 288, 0, 128), (2817, 3075, 64, 0, 128),
    (4001, 4095, 672, 0, 128),   # no 256x256 tile
    (75, 133, 70, 0, "general")])  # K % 32
def test_fp16_accumulation(monkeypatch, M, N, K, K2, want, layout):
    rows = np.r_[:5, 126:130, M // 2, M - 130:M - 126, M - 5:M] if M > 4000 else None
    check(monkeypatch, want, M, N, K, layout, K2, accum="f16", seed=M + 1, rows=rows)


def test_padding_past_k_is_not_read():
    """NaN and infinities in the storage past K, beside the partial last step."""
    M, N, K = 130, 140, 100
    A, B, _ = D.random_problem(69000, M, N, K)
    sA, sB = D.store(A, D.ROW, K + 5), D.store(B, D.COL, K + 5)
    sA[:, K:], sB[:, K:] = np.inf, np.nan
    got = gba.gemm_bias_act(torch.from_numpy(sA).cuda()[:, :K], torch.from_numpy(sB).cuda()[:, :K].t(),
                            act="none").cpu().numpy()
    U.assert_close(got, U.oracle_for(A, B, None, act=O.ACT_NONE), what="padding")
