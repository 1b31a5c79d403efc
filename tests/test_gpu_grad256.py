"""Backward pass of the 128 -> 256 -> 256 maps (back256_kernel, contract256_kernel, reduce256_kernel) where it can go wrong: a single
token block, both sides of a tile of 128 tokens, a last tile of fewer than four blocks, the degrees that are compiled in, absent biases,
projection layout, no softmax tokens, a batch (the sums go over it), more tiles than workgroups, so that a workgroup walks
from one head into the next and the products take its tiles in another order, and that together with several ranges of tiles per head.

Tolerance: the bars of test_gpu_value_distill_grad.py."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from oracle import value_distill_grad_oracle as G
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from tests.test_gpu_parity import oracle_map
from tests.test_gpu_value_distill_grad import GRAD_REL_L2, LOGIT_STD1, NAMES, bf16_representable, compare, round_io

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,N,P,R,dtype,layout,biases", (
    (1, 1, 2, 2, 2, "bf16", "bhnd", True),           # one linear token
    (1, 2, 127, 1, 3, "bf16", "bnhd", True),
    (2, 2, 129, 4, 4, "f32", "bnhd", True),
    (1, 1, 160, 8, 0, "bf16", "bhnd", True),         # a second tile of one block; no softmax tokens
    (2, 1, 385, 2, 2, "f32", "bhnd", False),
    (1, 1, 700, 1, 16, "f32", "bhnd", False),
    (2, 90, 257, 2, 2, "bf16", "bhnd", True),        # 540 query tiles: two per workgroup
))
def test_gradient(B, H, N, P, R, dtype, layout, biases):
    wl = W.replace(LOGIT_STD1, name=f"grad256_{B}_{H}_{N}_P{P}", B=B, H=H, N=N, dtype=dtype, d_hidden=256, d_feat=256, poly_degree=P,
                   seed=N + P)
    inp = bf16_representable(W.make_inputs(wl))
    if not biases:
        for m in (inp.phi_q, inp.phi_k):
            m.b1[:], m.b2[:] = 0, 0
    fq, fk = oracle_map(inp.phi_q), oracle_map(inp.phi_k)
    y = round_io(O.hybrid_attn(inp.q, inp.k, inp.v, None, None, 1, wl.scale), dtype)
    yh = round_io(O.hybrid_attn(inp.q, inp.k, inp.v, fq, fk, R, wl.scale), dtype)
    want = G.value_distill_grad(inp.q, inp.k, inp.v, fq, fk, R, wl.scale, sign_from=(y, yh))
    q, k, v, dq, dk = ha.to_device(inp)
    if not biases:
        dq, dk = (dataclasses.replace(m, b1=None, b2=None) for m in (dq, dk))
    den = np.empty((B, H, N))
    for b in range(B):
        for h in range(H):
            l = O.softmax_part(inp.q[b, h], inp.k[b, h], inp.v[b, h], R, wl.scale)[1]
            _, z = O.linear_state(inp.k[b, h], inp.v[b, h], fk, h, R)
            den[b, h] = l + O.feature_map(inp.q[b, h], fq, h) @ z
    put = lambda t: t if layout == "bhnd" else t.transpose(1, 2).contiguous().transpose(1, 2)
    to = lambda a: put(torch.from_numpy(a).to(device="cuda", dtype=q.dtype).contiguous())
    print(f"  case {wl.name} R={R} {dtype} {layout} biases={biases}", flush=True)
    _, gq, gk, _, _, _ = ha.hybrid_attn_value_distill_grad(put(q), put(k), put(v), dq, dk, R, wl.block_size, wl.scale, y_teacher=to(y),
                                                           teacher_is_cached=True, y_student=to(yh),
                                                           row_den=torch.from_numpy(den).to(device="cuda", dtype=torch.float32),
                                                           student_is_cached=True)
    torch.cuda.synchronize()
    assert compare(f"{wl.name}_R{R}_{dtype}_{layout}", (gq, gk), want) <= GRAD_REL_L2


@pytest.mark.parametrize("act,P,dtype", ((ha.HA_ACT_EXP, 1, "bf16"), (ha.HA_ACT_EXP, 4, "f32"), (ha.HA_ACT_EXP, 8, "bf16"),
                                         (ha.HA_ACT_RELU, 1, "f32"), (ha.HA_ACT_RELU, 4, "bf16"), (ha.HA_ACT_RELU, 8, "f32")))
def test_degrees_that_are_not_compiled_in(act, P, dtype):
    B, H, N, R = 1, 2, 300, 2
    wl = W.replace(LOGIT_STD1, name=f"grad256_act{act}_P{P}", B=B, H=H, N=N, dtype=dtype, d_hidden=256, d_feat=256, poly_degree=P, seed=P)
    check_heads(wl, R, act, "bhnd", range(H))


# 12 heads of 94 tiles over the queries and 71 over the keys: three and two tiles per workgroup of the passes, 9 + 6 + 6 and 12 + 9 ranges per
# head, images beyond the memory-side cache's share (non-temporal reads; cached ones never meet more than one tile per workgroup: 512 tiles
# are more than that share)
@pytest.mark.parametrize("act,P,dtype,layout", ((ha.HA_ACT_SOFTMAX, 2, "bf16", "bhnd"), (ha.HA_ACT_SOFTMAX, 4, "f32", "bnhd"),
                                                (ha.HA_ACT_EXP, 4, "bf16", "bnhd"), (ha.HA_ACT_RELU, 2, "f32", "bhnd")))
def test_several_ranges_and_tiles_per_workgroup(act, P, dtype, layout):
    H, N, R = 12, 12000, 4
    assert H * -(-N // 128) > 2 * 512 and H * -(-(N - N // R) // 128) > 512 and 256 // H >= 2 * 3
    wl = W.replace(LOGIT_STD1, name=f"grad256_long_act{act}_{dtype}", B=1, H=H, N=N, dtype=dtype, d_hidden=256, d_feat=256, poly_degree=P, seed=7)
    check_heads(wl, R, act, layout, (0, 6, 11))


def check_heads(wl, R, act, layout, heads):
    """The whole call on a teacher far from the student, so that no sign hangs on the outputs' rounding; the oracle takes a head at a time."""
    inp = bf16_representable(W.make_inputs(wl))
    fq, fk = oracle_map(inp.phi_q, act), oracle_map(inp.phi_k, act)
    q, k, v, dq, dk = ha.to_device(inp)
    dq.out_act = dk.out_act = act
    put = lambda t: t if layout == "bhnd" else t.transpose(1, 2).contiguous().transpose(1, 2)
    q, k, v = put(q), put(k), put(v)
    gen = torch.Generator(device="cuda").manual_seed(wl.seed)
    yt = put(torch.randn(q.shape, generator=gen, device="cuda").to(q.dtype))
    print(f"  case {wl.name} R={R} {wl.dtype} {layout}", flush=True)
    _, gq, gk, _, ys, _ = ha.hybrid_attn_value_distill_grad(q, k, v, dq, dk, R, wl.block_size, wl.scale, y_teacher=yt, teacher_is_cached=True)
    torch.cuda.synchronize()
    sign = torch.sign(ys.float() - yt.float())
    for h in heads:
        want = G.head_gradients_by_row_chunks(inp.q[0, h], inp.k[0, h], inp.v[0, h], fq, fk, h, R, wl.scale, sign=sign[0, h].cpu().numpy())
        pick = lambda g, ref: ({n: g[n][h] for n in NAMES}, dict(zip(NAMES, ref)))
        got_q, want_q = pick(gq, want[0])
        got_k, want_k = pick(gk, want[1])
        assert compare(f"{wl.name}_head{h}", (got_q, got_k), (want_q, want_k)) <= GRAD_REL_L2
