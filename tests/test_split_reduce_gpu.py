"""The library's own split of long reductions against the oracle: the partial
sums of every layout's split tile, added by the second kernel, at outputs
whose edge tiles are shifted, with every bias form, and the workspace zero
again afterwards."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2006_12645_amd import datagen as D
from paper_2006_12645_amd import gba

import gpu_util as U

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias_form", ["none", "row", "full"])
@pytest.mark.parametrize("layout", ["RR", "RC", "CR", "CC"])
@pytest.mark.parametrize("M,N,K,K2", [(64, 64, 16384, 0), (72, 200, 16392, 0), (104, 136, 16320, 136)])
def test_second_kernel(M, N, K, K2, layout, bias_form):
    print("CASE", M, N, K, K2, layout, bias_form, flush=True)
    la, lb = D.LAYOUT_NAMES[layout]
    A, B, row = D.random_problem(73000 + M, M, N, K)
    bias = {"none": None, "row": row, "full": D.uniform_f16(73500 + M, (M, N))}[bias_form]
    kw, okw = {}, {}
    if K2:
        P, Q, _ = D.random_problem(74000 + M, M, N, K2)
        kw.update(P=U.device_operand(P, la, 8), Q=U.device_operand(Q, lb, 8), second="sub")
        okw.update(second=-1, p_store=D.store(P, D.ROW), q_store=D.store(Q, D.COL), K2=K2)
    ws = torch.zeros(8 << 20, dtype=torch.uint8, device="cuda")
    dA, dB = U.device_operand(A, la, 8), U.device_operand(B, lb, 8)
    dbias = None if bias is None else torch.from_numpy(bias).cuda()
    outs = [gba.fused_gemm(dA, dB, bias=dbias, bias_op="sub", act="relu", workspace=w, **kw)
            for w in (ws, ws, "static")]
    torch.cuda.synchronize()
    assert not ws.any(), "workspace must be zero again"
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    if bias is not None:
        okw.update(bias=bias, bias_sign=-1)
    ref = O.fused(D.store(A, D.ROW), D.ROW, D.store(B, D.COL), D.COL, M, N, K, act=O.ACT_RELU, **okw)
    U.assert_close(outs[0].cpu().numpy(), ref, what=f"{M}x{N}x{K}+{K2} {layout}")
