"""Query kernel in two roles (small problems: phi_q beside the key loop) at the lengths of its key loop where the roles' barriers could
differ: no key block at all, one, odd and even, fewer and more than the map has pieces, the first with a separate loop of whole
blocks (33), both sides of the length from which fp32 calls take the other kernel (160 / 161), and longer ones; absent biases.

Tolerance: the bars of test_gpu_parity.py."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,N,R", ((64, 2, 200, 0), (128, 6, 40, 20), (64, 2, 66, 2), (128, 6, 385, 2), (128, 6, 960, 2), (64, 2, 1025, 4),
                                     (128, 6, 2050, 2), (64, 1, 2110, 2), (64, 1, 10240, 2), (64, 1, 10242, 2), (64, 1, 16384, 2), (64, 1, 16386, 2)))
@pytest.mark.parametrize("dtype", ("bf16", "f32"))
def test_lengths_of_the_key_loop(d, H, N, R, dtype):
    w = W.Workload(f"roles_d{d}_H{H}_N{N}_R{R}_{dtype}", 1, H, N, d, dtype, 128, R, d, d, poly_degree=2, seed=N + R)
    rows = np.unique(np.r_[0, 31, 32, 127, 128, N // 2, N - 2, N - 1]) if N > 600 else None
    check(w.name, W.make_inputs(w), rows=rows)


@pytest.mark.parametrize("d", (64, 128))
def test_absent_biases_and_row_denominators(d):
    """The denominators that a distillation step keeps come from this kernel too; with absent biases the map's are zeros."""
    w = W.Workload(f"roles_nobias_d{d}", 2, 3, 300, d, "f32", 64, 3, d, d, seed=d)
    inp = W.make_inputs(w)
    for m in (inp.phi_q, inp.phi_k):
        m.b1[:], m.b2[:] = 0, 0
    q, k, v, fq, fk = ha.to_device(inp)
    fq, fk = (dataclasses.replace(m, b1=None, b2=None) for m in (fq, fk))
    _, _, _, _, student, den = ha.hybrid_attn_value_distill_grad(q, k, v, fq, fk, w.R, 64, w.scale, y_teacher=torch.zeros_like(q), teacher_is_cached=True)
    torch.cuda.synchronize()
    maps = [O.FeatureMap(m.w1, m.b1, m.w2, m.b2, 2) for m in (inp.phi_q, inp.phi_k)]
    want = O.hybrid_attn(inp.q, inp.k, inp.v, *maps, w.R, w.scale)
    assert np.linalg.norm(student.cpu().numpy() - want) <= 5e-3 * np.linalg.norm(want)
    for b in range(2):
        for h in range(3):
            l = O.softmax_part(inp.q[b, h], inp.k[b, h], inp.v[b, h], w.R, w.scale)[1]
            z = O.linear_state(inp.k[b, h], inp.v[b, h], maps[1], h, w.R)[1]
            np.testing.assert_allclose(den[b, h].cpu().numpy(), l + O.feature_map(inp.q[b, h], maps[0], h) @ z, rtol=5e-3)
