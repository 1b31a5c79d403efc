"""The plain operator with more 128-query tiles than CUs: the instances of the query kernel that large calls run (8 waves a workgroup, or 4
with two workgroups per CU), with every activation, several degrees, absent biases, peaky and ever-rising logits, ragged lengths and strided
memory, at sizes that stay small because the heads are many and short.  All rows of a few heads against the fp64 oracle.

96 heads of 300 tokens are 288 tiles of 128 and 192 of 256 (8 waves, but for rate 1 at d = 128), 130 heads 260 of 256, whose second round is
nearly empty (4 waves); 128 heads of 500 tokens take 8 waves at rate 1 too.  Tolerance: the bars of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_guard_bands import run_forward
from test_gpu_parity import MAX_ABS, REL_L2, ROW_REL_L2, metrics, oracle_map, record, worst_row

pytestmark = pytest.mark.gpu

SHAPES = ((96, 300), (130, 300), (130, 259))            # heads, tokens: 8 waves; 4 waves; 4 waves, a last tile of three rows
RATE_1_SHAPES = SHAPES + ((128, 500),)
DTYPES = ("bf16", "f32")


def work(H, N, R, d=128, dtype="bf16", **kw):
    return W.Workload(f"many_d{d}_H{H}_N{N}_R{R}_{dtype}", 1, H, N, d, dtype, 128, R, d, d, seed=H + N + R, **kw)


def check_heads(inp, act=ha.HA_ACT_SOFTMAX, layout="bhnd", no_bias=(), heads=None):
    w = inp.workload
    q, k, v, fq, fk = ha.to_device(inp)
    fq.out_act = fk.out_act = act
    for which in no_bias:
        for fm, p in ((fq, inp.phi_q), (fk, inp.phi_k)):
            setattr(fm, which, None)
            getattr(p, which)[:] = 0
    if layout == "bnhd":
        q, k, v = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (q, k, v))
    assert w.H * -(-w.N // 128) > 256
    y = ha.hybrid_attn_forward(q, k, v, fq if w.R != 1 else None, fk if w.R != 1 else None, w.R, w.block_size, w.scale)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    for h in heads or (0, 1, w.H // 2, w.H - 1):
        ref = O.hybrid_attn_head(inp.q[0, h], inp.k[0, h], inp.v[0, h], oracle_map(inp.phi_q, act), oracle_map(inp.phi_k, act), h, w.R, w.scale)
        got = y[0, h].float().cpu().numpy()
        ma, rl = metrics(got, ref)
        wr, where = worst_row(got, ref)
        record(f"{w.name}_a{act}_P{w.poly_degree}_h{h}", ma, rl, row_rel_l2=wr)
        assert ma <= MAX_ABS and rl <= REL_L2 and wr <= ROW_REL_L2, (w.name, h, ma, rl, wr, where)


@pytest.mark.parametrize("H,N", SHAPES)
@pytest.mark.parametrize("d", (128, 64))
@pytest.mark.parametrize("dtype", DTYPES)
def test_rates(H, N, d, dtype):
    for R in (1, 2, 3, 4, 16) + ((0,) if d == 64 else ()):
        check_heads(W.make_inputs(work(H, N, R, d, dtype)), layout="bnhd" if R == 3 else "bhnd")


@pytest.mark.parametrize("H,N", SHAPES)
@pytest.mark.parametrize("d", (128, 64))
@pytest.mark.parametrize("P,act", ((1, 0), (2, 0), (4, 0), (8, 0), (1, 1), (2, 1), (1, 2), (2, 2)))
def test_degrees_and_activations(H, N, d, P, act):
    for dtype in DTYPES:
        check_heads(W.make_inputs(work(H, N, 4, d, dtype, poly_degree=P)), act=act, layout="bnhd" if P == 2 else "bhnd")


@pytest.mark.parametrize("H,N", SHAPES)
@pytest.mark.parametrize("d", (128, 64))
@pytest.mark.parametrize("no_bias", (("b1",), ("b2",), ("b1", "b2")))
def test_absent_biases(H, N, d, no_bias):
    for dtype in DTYPES:
        check_heads(W.make_inputs(work(H, N, 2, d, dtype)), no_bias=no_bias)


@pytest.mark.parametrize("H,N", RATE_1_SHAPES)
@pytest.mark.parametrize("d", (128, 64))
@pytest.mark.parametrize("kw", (dict(qk_gain=1.0), dict(qk_gain=4.0), dict(w_gain=8.0)), ids=("logit_std1", "peaky", "peaky_phi"))
@pytest.mark.parametrize("R", (1, 4))
def test_distributions(H, N, d, kw, R):
    kw = dict(kw)
    if "qk_gain" in kw:
        kw["qk_gain"] *= d ** 0.5
    check_heads(W.make_inputs(work(H, N, R, d, **kw)))


@pytest.mark.parametrize("H,N", RATE_1_SHAPES)
@pytest.mark.parametrize("d", (128, 64))
@pytest.mark.parametrize("R", (1, 2))
def test_every_key_raises_the_maximum(H, N, d, R):
    inp = W.make_inputs(work(H, N, R, d, qk_gain=2 * d ** 0.5))
    u = np.ones(d, dtype=np.float32) / np.sqrt(d)
    for h in (0, 1, H // 2, H - 1):
        inp.k[0, h] = inp.k[0, h][np.argsort(inp.k[0, h] @ u)]
        inp.q[0, h] = np.abs(inp.q[0, h])
    check_heads(inp)


@pytest.mark.parametrize("H,N", SHAPES)
@pytest.mark.parametrize("d,dtype,R", ((128, "bf16", 4), (64, "f32", 0), (128, "f32", 1)))
def test_writes_nothing_outside_its_buffers(H, N, d, dtype, R):
    run_forward(work(H, N, R, d, dtype))
