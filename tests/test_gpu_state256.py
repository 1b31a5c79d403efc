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


@pytest.mark.parametrize("width,H,N", ((256, 12, 3000), (128, 2, 3000), (128, 1, 20000), (384, 1, 12000)))
def test_workspace_without_the_query_sides_part(width, H, N):
    """The state tap runs the key side only: a workspace without the linear part's results (516 bytes per query and head)
    is enough, and nothing behind it is written."""
    w = W.Workload("s_ws", 1, H, N, 128, "bf16", 128, 4, width, width, poly_degree=3 if width == 384 else 2, seed=N)
    _, k, v, _, fk = ha.to_device(W.make_inputs(w))
    S, z = ha.hybrid_attn_linear_state(k, v, fk, 4)
    need = ha.hybrid_attn_workspace_bytes(ha.make_problem(k, 4, 128, 1.0), fk, fk)
    small = need - H * -(-N // 256) * 256 * 129 * 4 if width != 384 else need - H * -(-N // 32) * 32 * 128 * 4
    buf = torch.full((need,), 0x5a, dtype=torch.uint8, device="cuda")
    S2, z2 = ha.hybrid_attn_linear_state(k, v, fk, 4, workspace=buf[:small])
    torch.cuda.synchronize()
    assert torch.equal(S, S2) and torch.equal(z, z2)
    assert (buf[small:] == 0x5a).all()
