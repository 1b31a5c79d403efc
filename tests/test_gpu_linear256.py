"""The linear pass of the 128 -> 256 -> 256 maps on the query side (n = phi_q(q) S, e = phi_q(q) . z ahead of the query
kernel): against the fp64 oracle at the sizes where its tiles, its stream of operands and its rule on the tile size can
go wrong, every degree and activation, the denominators it takes part in, and the fixed workspace, where its results
are formed a part at a time.

Tolerance: the bars of test_gpu_parity.py; row denominators are fp32 sums over features rounded once to bf16
(<= 2^-9 each, random signs) plus softmax weights rounded likewise: 2e-3 relative."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check, oracle_map

pytestmark = pytest.mark.gpu


def work(N, B=1, H=2, R=4, dtype="bf16", P=2, seed=0):
    return W.Workload(f"l256_B{B}_H{H}_N{N}_R{R}_{dtype}_P{P}", B, H, N, 128, dtype, 128, R, 256, 256, poly_degree=P, seed=seed)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("B,H,N,R", (
    (1, 1, 5, 4), (1, 2, 33, 0), (2, 3, 128, 2), (1, 3, 129, 4),
    (1, 12, 5376, 4),            # 252 tiles of 256 queries: the small tile, 504 workgroups
    (1, 12, 5377, 16),           # 264 large tiles: workgroups of one and of two tiles, some across two heads
    (2, 100, 700, 0),            # 600 large tiles of 200 (batch, head) pairs: most workgroups change heads, a ragged last tile each
))
def test_sizes(B, H, N, R, dtype):
    w = work(N, B, H, R, dtype, seed=N)
    check(w.name, W.make_inputs(w), rows=W.sample_rows(w, n_random=16) if N > 600 else None)


@pytest.mark.parametrize("act", (ha.HA_ACT_SOFTMAX, ha.HA_ACT_EXP, ha.HA_ACT_RELU))
@pytest.mark.parametrize("P", (1, 2, 4, 8))
def test_degrees_and_activations(P, act):
    check("l256_act", W.make_inputs(work(600, P=P, R=3, seed=P)), act=act, layout="bnhd")


def test_row_denominators():
    inp = W.make_inputs(W.replace(work(1000, H=3, R=0, seed=5), qk_gain=128 ** 0.5))
    w = inp.workload
    q, k, v, fq, fk = ha.to_device(inp)
    _, _, _, _, y, den = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, 0, 128, w.scale, y_teacher=torch.zeros_like(q),
                                                           teacher_is_cached=True)
    torch.cuda.synchronize()
    assert torch.equal(ha.hybrid_attn_forward(q, k, v, fq, fk, 0, 128, w.scale), y)
    for h in range(w.H):
        z = O.feature_map(inp.k[0, h], oracle_map(inp.phi_k), h).sum(0)
        ref = O.feature_map(inp.q[0, h], oracle_map(inp.phi_q), h) @ z
        assert np.abs(den[0, h].double().cpu().numpy() - ref).max() <= 2e-3 * np.abs(ref).max()


@pytest.mark.parametrize("N", (1200, 4000, 8000))      # everything fits / results in the partials' place / in two parts
def test_fixed_workspace_gives_the_same_bits(N):
    w = work(N, H=12, seed=N)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    ref = ha.hybrid_attn_forward(q, k, v, fq, fk, w.R, 128, w.scale)
    out = torch.full_like(q, float("nan"))
    ha.hybrid_attn_forward_static(q, k, v, fq, fk, w.R, out, 128, w.scale)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


@pytest.mark.parametrize("P", (1, 2, 4))
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
def test_features_round_as_in_the_variants(P, dtype):
    """At rate 0 the last chunk of the chunk-causal variant sees what every query of the plain operator sees, through states
    that are summed in the same order; its epilogue evaluates phi_q tile by tile.  Same features, same bits."""
    w = work(1024, R=0, dtype=dtype, P=P, seed=11 + P)
    q, k, v, fq, fk = ha.to_device(W.make_inputs(w))
    plain = ha.hybrid_attn_forward(q, k, v, fq, fk, 0, 128, w.scale)
    causal = ha.hybrid_attn_forward(q, k, v, fq, fk, (0, 0, 256), 128, w.scale)
    torch.cuda.synchronize()
    assert torch.equal(plain[:, :, 768:], causal[:, :, 768:])
