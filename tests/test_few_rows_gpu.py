"""The few-row kernel against the oracle: requests of few rows, or of few
outputs over a reduction long enough that the library takes it from the
tiles, at the edges of its 16-row and 16/32/64-column blocks, its 64-deep
slabs (whole, partial, fewer than waves, one round of loads and more) and
odd leading dimensions.  The output is a window of a larger buffer whose
surroundings must stay untouched."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_12645_amd import datagen as D
from paper_2006_12645_amd import gba

import gpu_util as U

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(monkeypatch, M, N, K, layout, K2=0, second="sub", prologue=None, bias="full", bias_op="sub", act="none", pad=1,
          seed=0, blocks=None, rows=None):
    print("CASE", M, N, K, layout, K2, second, prologue, bias, act, pad, flush=True)
    A, B, row = D.random_problem(61000 + seed, M, N, K)
    b = {"row": row, "full": D.uniform_f16(62000 + seed, (M, N)), None: None}[bias]
    la, lb = D.LAYOUT_NAMES[layout]
    kw, okw = {}, {}
    if K2:
        P, Q, _ = D.random_problem(63000 + seed, M, N, K2)
        kw.update(P=U.device_operand(P, la, pad), Q=U.device_operand(Q, lb, pad), second=second)
        okw.update(second=1 if second == "add" else -1, p_store=D.store(P, D.ROW), q_store=D.store(Q, D.COL), K2=K2)
    if b is not None:
        kw.update(bias=U.misaligned(b) if pad % 2 else torch.from_numpy(b).cuda(), bias_op=bias_op)
        okw.update(bias=b, bias_kind=O.BIAS_ROW if b.ndim == 1 else O.BIAS_FULL, bias_sign=1 if bias_op == "add" else -1)
    else:
        okw.update(bias=None, bias_kind=O.BIAS_NONE)
    around = torch.full((M + 2, N + 3), 7.0, dtype=torch.float16, device="cuda")
    out = around[1:M + 1, 1:N + 1]
    with U.recorded_plans(monkeypatch) as plans:
        gba.fused_gemm(U.device_operand(A, la, pad), U.device_operand(B, lb, pad), prologue=prologue, act=act, out=out,
                       **kw)
    torch.cuda.synchronize()
    assert plans[0]["path"] == "few_rows" and blocks in (None, (plans[0]["bm"], plans[0]["bn"])), plans
    got = out.cpu().numpy()
    if rows is not None:
        got = got[rows]
        okw.update(rows=rows)
    ref = O.fused(D.store(A, D.ROW), D.ROW, D.store(B, D.COL), D.COL, M, N, K, prologue_relu=prologue == "relu",
                  act={"none": O.ACT_NONE, "relu": O.ACT_RELU, "tanh": O.ACT_TANH}[act], **okw)
    U.assert_close(got, ref, what=f"{M}x{N}x{K} {layout}")
    out.fill_(7.0)
    assert bool((around == 7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [
    (1, 64, 64, 0), (1, 65, 1, 0), (16, 33, 63, 65), (17, 96, 65, 0), (31, 130, 129, 7),
    (5, 48, 300, 520), (3, 1000, 515, 0), (16, 47, 1100, 0), (24, 4112, 600, 0),
    (7, 16473, 1100, 0), (20, 16473, 2100, 0),  # more columns than one round of any blocks covers
])
def test_fewer_rows_than_any_tile(monkeypatch, M, N, K, K2, layout):
    check(monkeypatch, M, N, K, layout, K2, prologue="relu" if K2 else None, seed=M + N + K)


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [
    (32, 264, 4096, 0),     # 16 waves, whole slabs
    (256, 256, 1544, 0),    # the last of one round of 16x16 workgroups (column-major B)
    (40, 2048, 2100, 264),  # 16x32 blocks, both products
])
def test_taken_from_the_tiles(monkeypatch, M, N, K, K2, layout):
    check(monkeypatch, M, N, K, layout, K2, second="add", prologue="relu" if K2 else None, bias="row", bias_op="add",
          act="relu", pad=8, seed=K)


@pytest.mark.parametrize("layout", ["RR", "CR"])
@pytest.mark.parametrize("M,N,blocks", [(64, 4096, (16, 64)), (72, 5416, (32, 64))])
def test_larger_blocks_of_row_major_b(monkeypatch, M, N, blocks, layout):
    check(monkeypatch, M, N, 3080, layout, bias="row", bias_op="add", act="relu", pad=8, seed=M, blocks=blocks,
          rows=np.r_[:3, 15:18, 31:34, 47:49, M - 10:M])


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [(64, 512, 16399, 0), (100, 100, 16400, 0), (65, 127, 9001, 8001)])
def test_long_reductions_outside_the_fast_path(monkeypatch, M, N, K, K2, layout):
    check(monkeypatch, M, N, K, layout, K2, prologue="relu" if K2 else None, bias="row", act="relu", seed=K)


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
def test_empty_reduction_is_the_bias(monkeypatch, layout):
    check(monkeypatch, 9, 80, 0, layout, bias="row", bias_op="sub", act="tanh")


@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,want", [(5, 75, 130, "few_rows"), (70, 75, 130, "unaligned")])
def test_largest_leading_dimension_of_32_bit_offsets(monkeypatch, M, N, K, want, layout):
    """Both kernels for requests outside the fast path address a tile with
    32-bit offsets up to leading dimensions of 2^23 - 1."""
    A, B, _ = D.random_problem(64500, M, N, K)
    ld = (1 << 23) - 1

    def far(x, row_major):
        x = torch.from_numpy(x if row_major else np.ascontiguousarray(x.T)).cuda()
        t = torch.empty(x.shape[0] * ld, dtype=torch.float16, device="cuda").view(x.shape[0], ld)[:, :x.shape[1]]
        t.copy_(x)
        return t if row_major else t.t()

    with U.recorded_plans(monkeypatch) as plans:
        got = gba.fused_gemm(far(A, layout[0] == "R"), far(B, layout[1] == "R"), act="none")
    assert plans[0]["path"] == want, plans
    U.assert_close(got.cpu().numpy(), U.oracle_for(A, B, None, act=O.ACT_NONE), what=layout)


def test_very_many_columns():
    """One row by 2.8e8 columns: as a launch of the few-row kernel 2^32 threads
    and more, which the runtime refuses."""
    N, K = 280_000_000, 8
    column = ((torch.arange(N, dtype=torch.int32, device="cuda") % 251 - 125).half() / 128)
    B = torch.empty((N, K), dtype=torch.float16, device="cuda")
    B.copy_(column[:, None])
    out = gba.gemm_bias_act(torch.full((1, K), 0.5, dtype=torch.float16, device="cuda"), B.t(), act="none")
    assert torch.equal(out[0], column * 4)


def test_infinite_operand_reaches_only_its_outputs():
    """Padding and clamped reads never mix: an infinity in one row of A or
    in B's storage past K changes no other output."""
    M, N, K = 7, 70, 100
    A, B, _ = D.random_problem(64000, M, N, K)
    dA, dB = U.device_operand(A, D.ROW, 5), U.device_operand(B, D.COL, 5)
    want = gba.gemm_bias_act(dA, dB, act="none").cpu().numpy()
    sA, sB = D.store(A, D.ROW, K + 5), D.store(B, D.COL, K + 5)
    sA[:, K:], sB[:, K:] = np.inf, np.nan
    sA[3, 50] = np.inf
    got = gba.gemm_bias_act(torch.from_numpy(sA).cuda()[:, :K], torch.from_numpy(sB).cuda()[:, :K].t(),
                            act="none").cpu().numpy()
    keep = [0, 1, 2, 4, 5, 6]
    assert np.array_equal(got[keep], want[keep])
    assert np.array_equal(got[3], np.where(B[50] > 0, np.inf, -np.inf).astype(np.float16))


def test_split_request_still_splits():
    """A request for a split across workgroups that the rule's tile can make
    keeps it (the same bits as on that tile, forced), where the few-row kernel
    would otherwise run; one that the rule's tile cannot make does not keep
    the few-row kernel away."""
    for M, N, K, splits in ((64, 512, 1536, 4), (64, 256, 4096, 1)):
        A, B, bias = D.random_problem(65000 + K, M, N, K)
        dA, dB, db = U.device_operand(A, D.ROW), U.device_operand(B, D.COL), torch.from_numpy(bias).cuda()
        t = gba.select_tile(M, N, K)
        d = gba.new_desc()
        d.layoutB, d.M, d.N, d.K = gba.GBA_COL_MAJOR, M, N, K
        d.A, d.lda, d.B, d.ldb = dA.data_ptr(), K, dB.data_ptr(), K
        d.C, d.ldc = dA.data_ptr(), N
        unsplit = gba.fused_plan(d)
        assert unsplit["path"] == "few_rows"
        d.split_k, d.workspace, d.workspace_bytes = 4, dA.data_ptr(), 1 << 30
        plain = gba.fused_plan(d)
        assert plain["splits"] == splits and (gba.workspace_size(d) > 0) == (splits > 1)
        got = gba.fused_gemm(dA, dB, bias=db, split=4)
        if splits > 1:
            assert torch.equal(got, gba.fused_gemm(dA, dB, bias=db, split=4, tile=t))
        else:
            assert plain == unsplit and torch.equal(got, gba.fused_gemm(dA, dB, bias=db))
        U.assert_close(got.cpu().numpy(), U.oracle_for(A, B, bias), what="split")
