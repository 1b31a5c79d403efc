"""State pass of the 128 -> 256 -> 256 maps, through the state tap, against the fp64 oracle: numbers of linear tokens around
the 128-token tile and the chunk, every rate's token map, dtypes, degrees and activations.

Tolerance: phi is rounded to bf16 (2^-9 relative) and V is bf16, sums are fp32: 2e-3 r.m.s. per term and less in the
sum; 5e-3 relative L2 leaves a factor of two (fp32 inputs are rounded to bf16 on load, another 2e-3 in phi)."""
import numpy as np
import pytest
import torch

from oracle import hybrid_attn_oracle as O
from paper_2509_24899_amd import hybrid_attn as ha
from paper_2509_24899_amd import workloads as W
from test_gpu_parity import oracle_map

pytestmark = pytest.mark.gpu


def state(N, R, B=1, H=2, dtype="bf16", P=2, act=ha.HA_ACT_SOFTMAX, seed=0):
    w = W.Workload("s256", B, H, N, 128, dtype, 128, R, 256, 256, poly_degree=P, seed=seed, qk_gain=3.0)
    inp = W.make_inputs(w)
    _, k, v, _, fk = ha.to_device(inp)
    fk.out_act = act
    S, z = ha.hybrid_attn_linear_state(k, v, fk, R)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            rs, rz = O.linear_state(inp.k[b, h], inp.v[b, h], oracle_map(inp.phi_k, act), h, R)
            for got, ref in ((S[b, h], rs), (z[b, h], rz)):
                got = got.double().cpu().numpy()
                assert np.isfinite(got).all()
                assert np.linalg.norm(got - ref) <= 5e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("dtype", ("bf16", "f32"))
@pytest.mark.parametrize("N,R", ((1, 0), (2, 2), (127, 0), (128, 0), (129, 0), (257, 2), (385, 3), (700, 4), (1025, 16), (900, 900)))
def test_token_counts(N, R, dtype):
    state(N, R, dtype=dtype, seed=N)


@pytest.mark.parametrize("P", (1, 2, 4, 8))
@pytest.mark.parametrize("act", (ha.HA_ACT_SOFTMAX, ha.HA_ACT_EXP, ha.HA_ACT_RELU))
def test_degrees_and_activations(P, act):
    state(500, 3, P=P, act=act, seed=P)


def test_several_tiles_per_chunk_and_more_heads_than_compute_units():
    state(5000, 4, B=2, H=12, seed=1)      # 10 chunks of 3 tiles per head, the last one ragged
    state(300, 2, B=3, H=100, seed=2)
