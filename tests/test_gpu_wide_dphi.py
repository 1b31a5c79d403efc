"""The first kernel of the wide maps' backward (dphi and the output activation), through the gradient call, where it can go
wrong: the last workgroup's idle waves (one token block, 7, 8 and 9 of them, a partly filled last one), a last block of
fewer than eight output tiles, each activation in its fused and two-pass form, both dtypes.

Tolerance: the bars of test_gpu_value_distill_grad.py."""
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from oracle import value_distill_grad_oracle as G
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from tests.test_gpu_parity import oracle_map
from tests.test_gpu_value_distill_grad import GRAD_REL_L2, LOGIT_STD1, bf16_representable, compare, round_io

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", (ha.HA_ACT_SOFTMAX, ha.HA_ACT_EXP, ha.HA_ACT_RELU))
@pytest.mark.parametrize("N,hid,feat,P,R,dtype", ((30, 256, 256, 2, 2, "bf16"), (224, 256, 128, 2, 2, "f32"),
                                                  (256, 128, 384, 3, 3, "bf16"), (257, 256, 256, 2, 2, "f32"),
                                                  (290, 384, 640, 4, 2, "bf16")))
def test_gradient(N, hid, feat, P, R, dtype, act):
    wl = W.replace(LOGIT_STD1, name=f"dphi_{N}_{hid}_{feat}", B=1, H=2, N=N, dtype=dtype, d_hidden=hid, d_feat=feat, poly_degree=P,
                   seed=N + feat)
    inp = bf16_representable(W.make_inputs(wl))
    fq, fk = oracle_map(inp.phi_q, act), oracle_map(inp.phi_k, act)
    y = round_io(O.hybrid_attn(inp.q, inp.k, inp.v, None, None, 1, wl.scale), dtype)
    yh = round_io(O.hybrid_attn(inp.q, inp.k, inp.v, fq, fk, R, wl.scale), dtype)
    want = G.value_distill_grad(inp.q, inp.k, inp.v, fq, fk, R, wl.scale, sign_from=(y, yh))
    q, k, v, dq, dk = ha.to_device(inp)
    dq.out_act = dk.out_act = act
    den = torch.empty((1, 2, N), dtype=torch.float32)
    for h in range(2):
        _, l, _ = O.softmax_part(inp.q[0, h], inp.k[0, h], inp.v[0, h], R, wl.scale)
        _, z = O.linear_state(inp.k[0, h], inp.v[0, h], fk, h, R)
        den[0, h] = torch.from_numpy(l + O.feature_map(inp.q[0, h], fq, h) @ z)
    print(f"  case {wl.name} {dtype} act={act}", flush=True)
    to = lambda a: torch.from_numpy(a).to(device="cuda", dtype=q.dtype).contiguous()
    _, gq, gk, _, _, _ = ha.hybrid_attn_value_distill_grad(q, k, v, dq, dk, R, wl.block_size, wl.scale, y_teacher=to(y),
                                                           teacher_is_cached=True, y_student=to(yh), row_den=den.cuda(),
                                                           student_is_cached=True)
    torch.cuda.synchronize()
    assert compare(f"{wl.name}_act{act}", (gq, gk), want) <= GRAD_REL_L2
