"""Purely linear attention (rate 0) with the 128-wide maps has a query-side kernel of its own: against the fp64 oracle at
the sizes where its split can go wrong (one row, one block, fewer blocks than waves or workgroups, one block past a
whole deal, more heads than CUs), every activation and degree, both dtypes, both layouts, and the denominators it
leaves for the gradient.

Tolerance: the bars of test_gpu_parity.py; row denominators are fp32 sums over features rounded once to bf16
(<= 2^-9 each, random signs): 2e-3 relative."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check, oracle_map

pytestmark = pytest.mark.gpu


def work(N, B=1, H=2, dtype="bf16", P=2, seed=0):
    return W.Workload(f"lin_B{B}_H{H}_N{N}_{dtype}_P{P}", B, H, N, 128, dtype, 128, 0, 128, 128, poly_degree=P, seed=seed)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("B,H,N", ((1, 1, 1), (1, 2, 31), (2, 3, 33), (1, 1, 256), (1, 1, 8193), (2, 12, 2600), (3, 100, 65)))
def test_sizes(B, H, N, dtype):
    check("lin", W.make_inputs(work(N, B, H, dtype, seed=N)))


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("B,H,N", ((1, 7, 97), (1, 32, 1526), (1, 129, 700), (4, 40, 1031), (3, 86, 300), (1, 257, 161)))
def test_pieces_on_the_eight_chiplets(B, H, N, dtype):
    """Workgroups are numbered chiplet by chiplet over pieces of heads: totals that are and are not multiples of eight, one
    workgroup per head (more than 128 heads), and more heads than CUs."""
    w = work(N, B, H, dtype, seed=N)
    check("lin_pieces", W.make_inputs(w), rows=np.unique(np.r_[0:N:53, N - 33:N]))


@pytest.mark.parametrize("act", (ha.HA_ACT_SOFTMAX, ha.HA_ACT_EXP, ha.HA_ACT_RELU))
@pytest.mark.parametrize("P", (1, 2, 4, 8))
def test_degrees_and_activations(P, act):
    # (exp and relu features are not normalised: their bars are those of the suite for these activations)
    check("lin_act", W.make_inputs(work(700, P=P, seed=P)), act=act, layout="bnhd")


def test_row_denominators():
    inp = W.make_inputs(W.replace(work(1000, H=3, seed=5), qk_gain=128 ** 0.5))
    w = inp.workload
    q, k, v, fq, fk = ha.to_device(inp)
    y_t = torch.zeros_like(q)
    _, _, _, _, y, den = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, 0, 128, w.scale, y_teacher=y_t, teacher_is_cached=True)
    torch.cuda.synchronize()
    fwd = ha.hybrid_attn_forward(q, k, v, fq, fk, 0, 128, w.scale)
    assert torch.equal(fwd, y)
    for h in range(w.H):
        z = O.feature_map(inp.k[0, h], oracle_map(inp.phi_k), h).sum(0)
        ref = O.feature_map(inp.q[0, h], oracle_map(inp.phi_q), h) @ z
        got = den[0, h].double().cpu().numpy()
        assert np.abs(got - ref).max() <= 2e-3 * np.abs(ref).max()
